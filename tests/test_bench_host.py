"""Host-side helpers of bench.py (no GPU): the comment-insensitive source
digest that keys the committed HBM counter summaries, the copy-calibrated
traffic read from them, and the one-GPU guard."""
import json
import os
import subprocess
import sys

import bench
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_code_text_ignores_comments_and_whitespace():
    a = "int f(int x) {  // doubles\n  return 2 * x; /* the\n multi-line */ }\n"
    b = "int f(int x) { return 2 * x; }"
    assert bench.code_text(a) == bench.code_text(b)
    assert bench.code_text(a) != bench.code_text(b.replace("2 * x", "3 * x"))


def test_source_digest_keeps_comment_edits_and_sees_code_edits(tmp_path):
    (tmp_path / "k.hip").write_text("__global__ void k(float* p) { p[0] = 1.f; }\n")
    (tmp_path / "h.h").write_text("// header\nconstexpr int kN = 4;\n")
    (tmp_path / "notes.txt").write_text("not a source")
    d0 = bench.source_digest(str(tmp_path))
    (tmp_path / "h.h").write_text("// a longer comment\n\nconstexpr int kN = 4;  // four\n")
    (tmp_path / "notes.txt").write_text("changed")
    assert bench.source_digest(str(tmp_path)) == d0
    (tmp_path / "h.h").write_text("constexpr int kN = 5;\n")
    assert bench.source_digest(str(tmp_path)) != d0


def test_counter_traffic_calibrates_and_rejects_stale_summaries(tmp_path, monkeypatch):
    data = {"source_sha256": bench.source_digest(), "unit": "launch",
            "copy": {"bytes_read": 1 << 20, "bytes_written": 1 << 20,
                     "fetch_kib": 512.0, "write_kib": 1024.0},
            "kernels": {"fwdbwd": {"fetch_kib": 100.0, "write_kib": 50.0, "calls": 3}}}
    path = tmp_path / "hbm_counters_{}.md"
    (tmp_path / "hbm_counters_x.md").write_text("# t\n\n```json\n" + json.dumps(data) + "\n```\n")
    monkeypatch.setattr(bench, "COUNTERS", str(path))
    # FETCH_SIZE counts half the copy's bytes (factor 2), WRITE_SIZE all (factor 1)
    assert bench.counter_traffic("x", "fwdbwd") == 100 * 1024 * 2 + 50 * 1024
    assert bench.counter_traffic("x", "update") is None
    assert bench.counter_traffic("missing", "fwdbwd") is None
    data["source_sha256"] = "0" * 64
    (tmp_path / "hbm_counters_x.md").write_text("```json\n" + json.dumps(data) + "\n```\n")
    assert bench.counter_traffic("x", "fwdbwd") is None


def test_model_counts_the_kernels_partials():
    """The partials of the dense gradients that the byte model prices: 21 slices
    of K + d columns for the wide preset (12 blocks of 128 columns on 256 CUs),
    32-window tiles for d 64 from 3,745 windows on, pairs of 16-window tiles for
    d 16, single ones below."""
    stress = workloads.PRESETS["stress"]
    assert bench.dense_parts(stress, stress.B) == (21, 256, stress.K + stress.d)
    poly, tiny = workloads.PRESETS["sweep_1024"], workloads.PRESETS["tiny"]
    for w, B, n in ((poly, 1024, 64), (poly, 3744, 234), (poly, 3745, 118), (poly, 5003, 157),
                    (poly, 65_536, 256), (tiny, 4096, 256), (tiny, 4097, 129), (tiny, 24_577, 193)):
        assert bench.dense_parts(w, B) == (n, n, w.K), (w.name, B)
    st = {"U": 1.0, "partials": 0.0, "long_rows": 0.0}
    m, over = bench.step_model(stress, stress.B, st, 2)
    assert over["wide_dw1"] == (21 * (stress.K + stress.d) - stress.K) * stress.H * 4
    assert m["wide_dw1"][2] == "mfma_split" and bench.step_model(poly, 1024, st, 0)[0]["fwdbwd"][2] == "mfma"
    assert bench.step_model(poly, 1024, st, 0)[0]["fwdbwd"][0] == 1024 * 3096 + poly.H * poly.K * 4


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr
