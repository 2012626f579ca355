"""Performance cases of the library: the calls that a user's program makes,
over the sizes that it makes them at.

A case is a dict of plain values.  ``kind`` says what is called:

  steps    Context.train_steps, S minibatches per call: the training loop of a
           program that has its next minibatches in device memory
  step     Context.train_step, one minibatch per call: minibatches that arrive
           one at a time
  score    Context.score: evaluation and serving
  gather   Context.gather: the window inputs on their own
  scatter  Context.scatter_add: float32 rows added into a table
  noalloc  scatter_add_noalloc: the same for short lists, without a context
  update   Context.scatter_update: the general op (storage format, id width,
           increment or assignment)

Model shapes are those of the workload presets and of the parity tests.  Word
ids follow a bounded Zipf law over a frequency-ranked vocabulary and corrupt
ids are uniform, as in the presets.  Parameters have the size of a model in the
middle of its training: pre-activations of a few tenths, so that tanh is not
the identity, and score differences of a few tenths, so that some windows meet
their margin and carry no gradient.  (Few margins lie within a rounding error
of zero, where two correct results may take different sides of the hinge.)  The
learning rate follows the convergence study's 0.25 sqrt(B / 16), held at 2.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1404_1521_amd as pg

# (d, win, H, largest V): the presets' shapes, then those of the parity tests
TINY = (16, 5, 8)
POLY = (64, 5, 32)
OTHER = [(64, 5, 64), (32, 7, 20), (112, 3, 48), (16, 31, 8)]
WIDE = [(128, 11, 256), (64, 3, 128), (192, 5, 192)]

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _model(name, kind, V, shape, B, S=1):
    d, win, H = shape
    return {"name": name, "kind": kind, "V": V, "d": d, "win": win, "H": H, "B": B, "S": S}


def _table(name, kind, rows, d, N, dtype="f32", op="inc", idx="i32", zipf=1.2):
    return {"name": name, "kind": kind, "rows": rows, "d": d, "N": N, "dtype": dtype, "op": op,
            "idx": idx, "zipf": zipf}


def listed():
    return [
        # the smallest model: a training loop bound by launches and latency
        _model("train-tiny", "steps", 1000, TINY, 32, 32),
        # one minibatch per call, as an online loop makes them
        _model("step-256", "step", 100_000, POLY, 256),
        # the headline minibatch
        _model("train-1024", "steps", 100_000, POLY, 1024, 16),
        # an ordinary larger minibatch that fills no tile or chunk evenly
        _model("train-5003", "steps", 100_000, POLY, 5003, 8),
        # the largest minibatch of the sweep
        _model("train-65536", "steps", 100_000, POLY, 65_536, 4),
        # a hidden layer at the limit of the fused kernel, not a preset's shape
        _model("train-h64-4096", "steps", 100_000, OTHER[0], 4096, 8),
        # the wide model with a vocabulary that no cache holds
        _model("train-wide-16384", "steps", 1_000_000, WIDE[0], 16_384, 2),
        # a held-out set scored in one call
        _model("score-8192", "score", 100_000, POLY, 8192),
        # the inputs of a large minibatch of the wide model
        _model("gather-16384", "gather", 1_000_000, WIDE[0], 16_384),
        # the scatter-add on its own: 65,536 windows of five rows
        _table("scatter-327680", "scatter", 100_000, 64, 327_680),
        # the general op on a 16-bit table, ids as torch makes them
        _table("update-bf16-327680", "update", 100_000, 64, 327_680, "bf16", "inc", "i64"),
        # rows of an odd count replaced
        _table("set-f16-20011", "update", 50_000, 100, 20_011, "f16", "set", "i64", 1.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "step", "score", "gather", "scatter", "noalloc",
                       "update", "update"])
    if kind in ("steps", "step", "score", "gather"):
        group = rng.choice(["preset", "preset", "other", "wide"])
        if group == "preset":
            shape, most = rng.choice([POLY, POLY, POLY, TINY]), 65_536
        elif group == "other":
            shape = rng.choice(OTHER)
            most = 200_000 // (shape[1] + 1)
        else:
            shape, most = rng.choice(WIDE), 16_384
        B = _log(rng, 8, most)
        V = _log(rng, 1000, 100_000 if group != "wide" else 500_000)
        S = 1 if kind != "steps" else max(1, min(rng.randint(2, 16), 2 * most // B))
        c = _model("", kind, V, shape, B, S)
    else:
        d = rng.choice([16, 32, 48, 64, 100, 128, 200, 256])
        N = _log(rng, 50, 8192 if kind == "noalloc" else 60_000_000 // (d + 32))
        rows = _log(rng, 500, 300_000)
        dtype, op, idx = "f32", "inc", "i32"
        if kind == "update":
            dtype, op = rng.choice(["f32", "bf16", "bf16", "f16"]), rng.choice(["inc", "inc", "set"])
            idx = rng.choice(["i32", "i64"])
            d = rng.choice([d, d, d + rng.randint(-15, 0)])  # widths of every alignment
        c = _table("", kind, rows, d, N, dtype, op, idx, rng.choice([0.0, 1.0, 1.2]))
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

_CDF: dict = {}
_STREAM = None


def _stream():
    """The program's one stream (a stream of its own, so that multi-step calls
    are recorded into a graph)."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def _zipf(gen, n, s, shape):
    """Bounded Zipf(s) ids over [0, n), id = rank - 1, by inverse CDF (s = 0: uniform)."""
    key = (n, s)
    if key not in _CDF:
        if len(_CDF) > 8:
            _CDF.clear()
        c = torch.arange(1, n + 1, dtype=torch.float64, device="cuda").pow_(-s).cumsum_(0)
        _CDF[key] = c.div_(c[-1].clone())
    u = torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen)
    return torch.searchsorted(_CDF[key], u, right=True).clamp_(max=n - 1)


def _lr(B):
    return min(2.0, 0.25 * math.sqrt(B / 16.0))


def _model_inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    V, d, win, H, B, S = c["V"], c["d"], c["win"], c["H"], c["B"], c["S"]
    K = win * d

    def normal(std, *shape):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=gen)

    params = {"E": normal(0.3, V, d), "W1": normal(1.5 / math.sqrt(K), H, K), "b1": normal(0.1, H),
              "w2": normal(1.5 / math.sqrt(H), H), "b2": normal(0.1, 1)}
    lead = (S, B) if c["kind"] == "steps" else (B,)
    windows = _zipf(gen, V, 1.0, lead + (win,)).to(torch.int32)
    corrupt = torch.randint(0, V, lead, device="cuda", generator=gen, dtype=torch.int32)
    return params, windows, corrupt


def _table_inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[c["dtype"]]
    table = torch.empty(c["rows"], c["d"], device="cuda").normal_(0.0, 0.01, generator=gen).to(dt)
    idx = _zipf(gen, c["rows"], c["zipf"], (c["N"],))
    idx = idx if c["idx"] == "i64" else idx.to(torch.int32)
    Y = torch.empty(c["N"], c["d"], device="cuda").normal_(0.0, 1e-3, generator=gen).to(dt)
    return table, idx, Y


def prepare(c, seed):
    kind = c["kind"]
    if kind in ("steps", "step", "score", "gather"):
        params, windows, corrupt = _model_inputs(c, seed)
        s = {"kind": kind, "params": params, "windows": windows, "corrupt": corrupt,
             "lr": _lr(c["B"]),
             "ctx": pg.Context(c["V"], c["d"], c["win"], c["H"], max_batch=c["B"],
                               stream=_stream())}
        if kind in ("steps", "step"):
            s["losses"] = torch.zeros(c["S"], device="cuda")
        elif kind == "score":
            s["out"] = torch.empty(c["B"], device="cuda")
        else:
            s["X"] = torch.empty(c["B"], c["win"] * c["d"], device="cuda")
            s["Xc"] = torch.empty(c["B"], c["d"], device="cuda")
    else:
        table, idx, Y = _table_inputs(c, seed)
        s = {"kind": kind, "table": table, "idx": idx, "Y": Y,
             "op": pg.OP_SET if c["op"] == "set" else pg.OP_INC}
        if kind == "noalloc":
            s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
            s["stream"] = _stream()
        else:  # a context for the op alone: the model shape is the smallest
            s["ctx"] = pg.Context(1000, 16, 5, 8, max_batch=1, max_scatter=c["N"],
                                  max_rows=c["rows"], stream=_stream())
    torch.cuda.synchronize()  # inputs were made on torch's stream, the calls run on the context's
    return s


def run(s):
    kind = s["kind"]
    if kind == "steps":
        s["ctx"].train_steps(s["params"], s["windows"], s["corrupt"], s["lr"], s["losses"])
        return {"losses": s["losses"], **s["params"]}
    if kind == "step":
        s["ctx"].train_step(s["params"], s["windows"], s["corrupt"], s["lr"], s["losses"])
        return {"losses": s["losses"], **s["params"]}
    if kind == "score":
        return s["ctx"].score(s["params"], s["windows"], s["out"])
    if kind == "gather":
        return s["ctx"].gather(s["params"]["E"], s["windows"], s["corrupt"], s["X"], s["Xc"])
    if kind == "scatter":
        s["ctx"].scatter_add(s["table"], s["idx"], s["Y"])
    elif kind == "noalloc":
        pg.scatter_add_noalloc(s["table"], s["idx"], s["Y"], status=s["status"],
                               stream=s["stream"])
        return {"table": s["table"], "status": s["status"]}
    else:
        s["ctx"].scatter_update(s["table"], s["idx"], s["Y"], op=s["op"])
    return s["table"]


# ------------------------------------------------------------------ what a pass needs

def _distinct(n, s, draws, uniform_draws=0):
    """Expected distinct ids of `draws` Zipf(s) and `uniform_draws` uniform ids over [0, n)."""
    p = np.arange(1, n + 1, dtype=np.float64) ** -s
    p /= p.sum()
    miss = draws * np.log1p(-np.minimum(p, 1 - 1e-12))
    if n > 1:
        miss = miss + uniform_draws * math.log1p(-1.0 / n)
    return float(np.sum(-np.expm1(miss)))


def work(c):
    kind = c["kind"]
    if kind in ("steps", "step", "score", "gather"):
        d, win, H, B, S, V = c["d"], c["win"], c["H"], c["B"], c["S"], c["V"]
        K = win * d
        dense = 4 * (H * K + 2 * H + 1)
        if kind == "score":
            return {"bytes": 4 * B * win + 4 * d * _distinct(V, 1.0, B * win) + dense + 4 * B,
                    "flops": 2.0 * B * H * K}
        rows = _distinct(V, 1.0, B * win, B)
        if kind == "gather":
            return {"bytes": 4.0 * B * (win + 1) * (1 + d) + 4 * d * rows, "flops": 0.0}
        # forward of x and of the centre block's copy, dW1 of both, one gradient row per entry
        flops = B * (4.0 * H * K + 4.0 * H * d + (win + 1) * 2.0 * H * d)
        return {"bytes": S * (4.0 * B * (win + 1) + 2 * 4 * d * rows + 2 * dense + 4),
                "flops": S * flops}
    es = 4 if c["dtype"] == "f32" else 2
    ib = 8 if c["idx"] == "i64" else 4
    N, d = c["N"], c["d"]
    rows = _distinct(c["rows"], c["zipf"], N)
    if c["op"] == "set":  # the last entry of a row is all that has to be read of Y
        return {"bytes": ib * N + 2.0 * rows * d * es, "flops": 0.0}
    return {"bytes": ib * N + float(N) * d * es + 2.0 * rows * d * es, "flops": 2.0 * N * d}


def tolerance(c):
    kind = c["kind"]
    if kind == "gather" or c.get("op") == "set":
        return "exact"  # copies
    # about four times the error measured against 64 bits: 3.2e-7 at most after
    # 32 steps (b1; 1.1e-7 after 16), 2.4e-7 for scores
    if kind in ("steps", "step"):
        return {"rel": 1.5e-6}
    if kind == "score":
        return {"rel": 1e-6}
    # increments: one rounding of each row to its format (bf16: 9e-4 measured,
    # over touched and untouched rows), and float32 sums (3.9e-8 measured; the
    # hot rows of a short table add up more entries)
    return {"rel": {"f32": 4e-7, "bf16": 4e-3, "f16": 5e-4}[c["dtype"]]}


# ------------------------------------------------------------------ 64-bit results

def _exact_steps(c, seed):
    params, windows, corrupt = _model_inputs(c, seed)
    P = {k: v.double() for k, v in params.items()}
    d, win, B, S = c["d"], c["win"], c["B"], c["S"]
    mid, lr = win // 2, _lr(B)
    losses = []
    for s in range(S):
        w = (windows[s] if c["kind"] == "steps" else windows).long()
        q = (corrupt[s] if c["kind"] == "steps" else corrupt).long()
        x = P["E"][w]                          # B, win, d
        xt = x.clone()
        xt[:, mid] = P["E"][q]
        x, xt = x.reshape(B, -1), xt.reshape(B, -1)
        h, ht = torch.tanh(x @ P["W1"].T + P["b1"]), torch.tanh(xt @ P["W1"].T + P["b1"])
        margin = 1.0 - h @ P["w2"] + ht @ P["w2"]
        on = (margin > 0).double() / B
        losses.append((margin.clamp(min=0)).mean())
        dz = -on[:, None] * P["w2"] * (1 - h * h)
        dzt = on[:, None] * P["w2"] * (1 - ht * ht)
        gx, gxt = (dz @ P["W1"]).reshape(B, win, d), (dzt @ P["W1"]).reshape(B, win, d)
        both = gx + gxt
        both[:, mid] = gx[:, mid]
        grads = {"W1": dz.T @ x + dzt.T @ xt, "b1": (dz + dzt).sum(0),
                 "w2": (on[:, None] * (ht - h)).sum(0)}
        P["E"].index_add_(0, w.reshape(-1), both.reshape(-1, d), alpha=-lr)
        P["E"].index_add_(0, q, gxt[:, mid].contiguous(), alpha=-lr)
        for k, g in grads.items():
            P[k] -= lr * g
    return {"losses": torch.stack(losses), **P}


def exact(c, seed):
    kind = c["kind"]
    if kind in ("steps", "step"):
        return _exact_steps(c, seed)
    if kind in ("score", "gather"):
        params, windows, corrupt = _model_inputs(c, seed)
        if kind == "gather":
            E = params["E"]
            return (E[windows.long()].reshape(c["B"], -1).double(), E[corrupt.long()].double())
        P = {k: v.double() for k, v in params.items()}
        x = P["E"][windows.long()].reshape(c["B"], -1)
        return torch.tanh(x @ P["W1"].T + P["b1"]) @ P["w2"] + P["b2"]
    table, idx, Y = _table_inputs(c, seed)
    out, idx = table.double(), idx.long()
    if c["op"] == "set":
        last = torch.full((c["rows"],), -1, device="cuda", dtype=torch.int64)
        last.scatter_reduce_(0, idx, torch.arange(c["N"], device="cuda"), "amax")
        rows = torch.nonzero(last >= 0).reshape(-1)
        out[rows] = Y[last[rows]].double()
    else:
        out.index_add_(0, idx, Y.double())
    return {"table": out, "status": None} if kind == "noalloc" else out
