// Fused gather + forward + hinge + backward for compile-time shapes, one
// workgroup of 16 waves per group of consecutive 16-window tiles (16x16x4 f32
// MFMA), ending in the per-entry embedding gradient rows G.
//
// Per tile of 16 windows (rows r), with V = dz + dz~, dz or dz~ (per window,
// H values each):
//   X         the tile's embedding rows -- positions 0..win-1 and the
//             corrupt row as position win -- staged in LDS once, laid out
//             [position][column quad][window] so that both MFMA operand
//             layouts read it without bank conflicts; the rows of the next
//             pair are loaded into registers while a pair computes, and the
//             ids of the pair after it at the same time;
//   forward   Z = X W1^T: wave w takes hidden block nt = w % NT and the
//             K-chunks kc = w / NT + (16 / NT) i; the corrupted copy only
//             differs in block c, so z~ = z - zctr + zcor (§1 model, x~);
//   epilogue  tanh, both scores, hinge mask, dz, dz~ and their sum; a lane
//             of waves 0-7 takes one hidden unit of one row;
//   dW1       dW1 += V^T X for the wave's (nt, chunks), held in registers
//             across the workgroup's tiles and written once as its partial;
//   G         G[e][:] = W1_j^T V for entry e = b(win+1) + j: context
//             positions take dz + dz~, the true centre dz, the corrupt entry
//             (j = win) dz~ through block c; 16x16 output tiles (position,
//             16 columns) round-robin over the waves.
// W1 is staged once per workgroup in LDS (row stride K + 4 floats, rows
// >= H zero) and read from there as the B operand of the forward and of G.
// Small batches (one tile per workgroup, CUs to spare) split the backward:
// two workgroups take the same tile, both run the forward and the epilogue,
// and each computes half of the dW1 and G output tiles, writing its own
// dense-partial slot.
// TP is the tiles of a phase: 1 where a workgroup has a single tile, three
// barriers; 2 where it has more, tiles in pairs, four barriers per pair: each
// phase holds the work of both tiles (two independent MFMA chains per wave, and
// every wave busy in the epilogue), at the price of a single X buffer.
#pragma once
#include "common.h"
#include "launch.h"

namespace pg {

__device__ __forceinline__ f4 mfma16x4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, int WIN, int NT, int TP>
struct F8Shape {
  static constexpr int HP = NT * 16;         // hidden units, padded
  static constexpr int K = D * WIN;          // window vector length
  static constexpr int C = WIN / 2;          // centre position
  static constexpr int W1P = WIN + 1;        // positions incl. the corrupt row
  static constexpr int DQ = D / 16;          // 16-column chunks per row
  static constexpr int QD = D / 4;           // column quads per row
  static constexpr int NCH = K / 16;         // K-chunks
  static constexpr int KW = kF8Waves / NT;   // dW1: waves per hidden block
  static constexpr int CPW = (NCH + KW - 1) / KW;  // dW1: chunks per wave
  static constexpr int KWF = kF8Waves / (TP * NT);  // forward: waves per output tile
  static constexpr int CPWF = (NCH + KWF - 1) / KWF;  // forward: chunks per wave
  static constexpr int NGT = W1P * DQ;       // G output tiles per 16-window tile
  static constexpr int GPW = (TP * NGT + kF8Waves - 1) / kF8Waves;  // G tiles per wave
  static constexpr int XF1 = W1P * QD * kTileRows;  // float4 pieces of X per tile
  static constexpr int XF4 = TP * XF1;              // ... per group of TP tiles
  static constexpr int XPT = (XF4 + kF8Threads - 1) / kF8Threads;  // pieces per thread
  static constexpr int S = K + 4;            // W1 row stride in LDS
  // LDS, in floats
  static constexpr int kW1 = HP * S;
  static constexpr int kX = XF4 * 4;                       // X
  static constexpr int kZp = kF8Waves * 3 * 4 * kWave;     // forward split-K partials
  static constexpr int kVt = TP * 3 * kTileRows * (HP + 1);
  static constexpr int kRed = kF8Waves * (2 * HP + 2);
  static constexpr int kLds = kW1 + kX + kZp + kVt + kRed;
  static_assert(D % 16 == 0 && WIN % 2 == 1 && kF8Waves % (TP * NT) == 0, "shape");
  static_assert(kLds * 4 <= 160 * 1024, "LDS of one workgroup");
  static_assert(HP <= 32, "one hidden unit per lane of each 32-lane row half");
};

template <int D, int WIN, int NT, int TP, int NH>
__device__ void fwdbwd8_wg(const FwdArgs& a, int wg, float* lds) {
  using Sh = F8Shape<D, WIN, NT, TP>;
  constexpr int HP = Sh::HP, K = Sh::K, C = Sh::C, W1P = Sh::W1P, DQ = Sh::DQ, QD = Sh::QD;
  constexpr int NCH = Sh::NCH, CPW = Sh::CPW, NGT = Sh::NGT, GPW = Sh::GPW;
  constexpr int KWF = Sh::KWF, CPWF = Sh::CPWF;
  constexpr int XF1 = Sh::XF1, XF4 = Sh::XF4, XPT = Sh::XPT, S = Sh::S;
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);  // wave-uniform
  const int n16 = lane & 15, g = lane >> 4;
  // forward: this wave's output tile otf (tile otf / NT of the group, hidden
  // block otf % NT) and chunk set kqf
  const int otf = w % (TP * NT), kqf = w / (TP * NT);
  const int tpf = otf / NT, ntf = otf % NT;

  float* w1s = lds;                       // [HP][K+4]
  float* xl = w1s + Sh::kW1;              // [TP][W1P][QD][16] float4
  float* zp = xl + Sh::kX;                // [kqf][3][otf][4][64]
  float* vt = zp + Sh::kZp;               // [TP][3][16][HP+1]
  float* red = vt + Sh::kVt;              // [waves][2*HP+2]

  // Split backward (NH == 2): workgroups 2q and 2q+1 take the same
  // tiles, both run the forward and the epilogue, and half h = wg & 1 takes
  // every second dW1 output tile and every second G output tile (linear
  // indices L = 2 (w + 16 i) + h); each writes its own partial slot, and the
  // db1 / dw2 / loss sums come from half 0 only.
  static_assert(NH == 1 || (NH == 2 && TP == 1), "the split takes single-tile workgroups");
  constexpr int nh = NH;
  const int h = wg & (nh - 1);
  const int tile0 = (wg / nh) * a.tiles_per_wg;
  // dW1 output tiles L = kc NT + nt of this wave: L = nh (w + 16 i) + h, all
  // in hidden block ntd
  constexpr int NLT = NCH * NT;
  const int ntd = (nh * w + h) % NT;
  const int ntl = min(a.tiles_per_wg, a.ntiles - tile0);  // tiles of this workgroup (>= 1)

  // ids of the X pieces of this thread in the group of TP tiles starting at
  // `tile`: piece pi = t + 1024 p covers tile pi / XF1 of the group and,
  // with q = pi % XF1, window r = q % 16, column quad (q / 16) % QD,
  // position q / (16 QD) (position win: the corrupt id).  Rows >= B read
  // row 0.  The loads are only issued here: the range check waits for them,
  // so it sits in load_x, where the rows' addresses need the ids anyway.
  auto load_ids = [&](int tile, int32_t (&id)[XPT]) {
#pragma unroll
    for (int p = 0; p < XPT; ++p) {
      const int pi = t + kF8Threads * p;
      const int tp = pi / XF1, q = pi - tp * XF1;
      const int r = q % kTileRows, j = q / (kTileRows * QD);
      const int b = (tile + tp) * kTileRows + r;
      id[p] = 0;
      if (pi < XF4 && b < a.B) id[p] = (j < WIN) ? a.windows[(size_t)b * WIN + j] : a.corrupt[b];
    }
  };
  // the rows of one tile into registers; an id outside [0, V) reads row 0
  // and raises the flag (after every load is issued)
  auto load_x = [&](const int32_t (&id)[XPT], f4 (&xr)[XPT]) {
    bool bad = false;
#pragma unroll
    for (int p = 0; p < XPT; ++p) {
      const int pi = t + kF8Threads * p;
      const int qq = ((pi % XF1) / kTileRows) % QD;
      const bool bk = (uint32_t)id[p] >= (uint32_t)a.V;
      bad |= bk;
      xr[p] = pi < XF4 ? ld4(a.E + (size_t)(bk ? 0 : id[p]) * D + 4 * qq) : kZero4;
    }
    if (bad) atomicOr(a.flag, kFlagBadId);
  };
  auto store_x = [&](const f4 (&xr)[XPT]) {
#pragma unroll
    for (int p = 0; p < XPT; ++p) {
      const int pi = t + kF8Threads * p;
      if (pi < XF4) st4(xl + 4 * pi, xr[p]);
    }
  };
  // ---- prologue: ids of the first tile, W1 and the first tile's rows in
  // flight together (the rows wait only for the ids), then the ids of the
  // second pair
  int32_t ids[XPT], idn[XPT];
  f4 xr[XPT];
  load_ids(tile0, ids);
  {  // W1 into LDS (rows >= H zero); loads batched before the stores
    constexpr int N4 = HP * (K / 4);
    constexpr int U = (N4 + kF8Threads - 1) / kF8Threads;
    f4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = u * kF8Threads + t;
      const int n = i / (K / 4), k4 = i - n * (K / 4);
      v[u] = (i < N4 && n < a.H) ? ld4(a.W1 + (size_t)n * K + 4 * k4) : kZero4;
    }
    load_x(ids, xr);
    if (TP == 2 && ntl > TP) load_ids(tile0 + TP, idn);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = u * kF8Threads + t;
      const int n = i / (K / 4), k4 = i - n * (K / 4);
      if (i < N4) st4(w1s + n * S + 4 * k4, v[u]);
    }
  }
  // epilogue lane map: hidden unit hn = lane % 32 of row 2w + lane / 32
  const int hn = lane & 31, rsel = lane >> 5;
  const float b1v = hn < a.H ? a.b1[hn] : 0.f;
  const float w2v = hn < a.H ? a.w2[hn] : 0.f;
  const float b2v = a.b2[0];

  f4 accW[CPW];
#pragma unroll
  for (int ci = 0; ci < CPW; ++ci) accW[ci] = kZero4;
  float db1a = 0.f, dw2a = 0.f, lossa = 0.f;

  // ---- forward of the tiles in X: split-K partials into zp
  auto forward = [&](const float* Xg) {
    // ---- forward: wave (otf, kqf) over chunks kc = kqf + KWF ci; common
    // blocks, true centre and corrupt centre accumulate separately
    const float* X = Xg + 4 * XF1 * tpf;
    f4 zc = kZero4, zctr = kZero4, zcor = kZero4;
#pragma unroll
    for (int ci = 0; ci < CPWF; ++ci) {
      const int kc = kqf + KWF * ci;
      if (kc < NCH) {
        const int j = kc / DQ, qq = 4 * (kc % DQ) + g;
        const f4 xa = ld4(X + 4 * ((j * QD + qq) * kTileRows + n16));
        const f4 wb = ld4(w1s + (ntf * 16 + n16) * S + kc * 16 + 4 * g);
        if (j != C) {
#pragma unroll
          for (int q = 0; q < 4; ++q) zc = mfma16x4(xa[q], wb[q], zc);
        } else {
          const f4 xt = ld4(X + 4 * ((WIN * QD + qq) * kTileRows + n16));
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            zctr = mfma16x4(xa[q], wb[q], zctr);
            zcor = mfma16x4(xt[q], wb[q], zcor);
          }
        }
      }
    }
    // partials [kqf][type][otf][component][lane] (component-major: a
    // reader of one component of every lane touches consecutive words)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      zp[(((kqf * 3 + 0) * (TP * NT) + otf) * 4 + i) * kWave + lane] = zc[i];
      zp[(((kqf * 3 + 1) * (TP * NT) + otf) * 4 + i) * kWave + lane] = zctr[i];
      zp[(((kqf * 3 + 2) * (TP * NT) + otf) * 4 + i) * kWave + lane] = zcor[i];
    }
  };
  // ---- epilogue of the tiles starting at row0: zp -> V (vt) and the
  // accumulators
  auto epilogue = [&](int row0) {
    // ---- epilogue: lane (hn, rsel) of wave w < 8 TP takes hidden unit hn of
    // row 2w + rsel of the group (tile tp = r / 16, row rr = r % 16 in it)
    if (w < TP * kTileRows / 2) {
      const int r = 2 * w + rsel;
      const int row = row0 + r;
      const int tp = r / kTileRows, rr = r % kTileRows;
      const int ot = tp * NT + (hn >> 4), src = (hn & 15) + 16 * (rr >> 2), comp = rr & 3;
      float Zc = 0.f, Zctr = 0.f, Zcor = 0.f;
      if (hn < HP) {
#pragma unroll
        for (int v = 0; v < KWF; ++v) {
          Zc += zp[(((v * 3 + 0) * (TP * NT) + ot) * 4 + comp) * kWave + src];
          Zctr += zp[(((v * 3 + 1) * (TP * NT) + ot) * 4 + comp) * kWave + src];
          Zcor += zp[(((v * 3 + 2) * (TP * NT) + ot) * 4 + comp) * kWave + src];
        }
      }
      const float z = b1v + (Zc + Zctr);
      const float zt = b1v + (Zc + Zcor);
      const float h = tanh_fast(z), ht = tanh_fast(zt);
      // h - h~ = tanh(z - z~) (1 - h h~), z - z~ = zctr - zcor without
      // cancellation against the common part
      const float hmh = tanh_fast(Zctr - Zcor) * (1.f - h * ht);
      float ps = w2v * h, pst = w2v * ht;
#pragma unroll
      for (int o = 1; o < 32; o <<= 1) {
        ps += __shfl_xor(ps, o);
        pst += __shfl_xor(pst, o);
      }
      const float mg = 1.f - (b2v + ps) + (b2v + pst);
      const bool on = row < a.B && mg > 0.f;  // hinge active (derivative 0 at margin 0)
      const float gst = on ? a.invB : 0.f;    // d loss/d s~ = m/B, d loss/d s = -m/B
      const float gw = gst * w2v;
      const float dz = -gw * (1.f - h * h);
      const float dzt = gw * (1.f - ht * ht);
      const float dsum = gw * hmh * (h + ht);  // dz + dz~ = g w2 (h - h~)(h + h~)
      if (hn < HP) {
        vt[((tp * 3 + 0) * kTileRows + rr) * (HP + 1) + hn] = dsum;
        vt[((tp * 3 + 1) * kTileRows + rr) * (HP + 1) + hn] = dz;
        vt[((tp * 3 + 2) * kTileRows + rr) * (HP + 1) + hn] = dzt;
      }
      db1a += dsum;
      dw2a -= gst * hmh;  // -(m/B) h + (m/B) h~
      if (hn == 0) lossa += on ? mg : 0.f;
    }
  };
  // ---- dW1 and G of the tiles in X starting at row0 (reads vt)
  auto backward = [&](const float* Xg, int row0) {
    // ---- dW1 += V^T X for this wave's output tiles (block ntd, chunks kc),
    // the group's tiles in order.  A operand: lane (n16, g) holds
    // V[4ii+g][ntd*16 + n16]; B operand: X[4ii+g][16kc + n16].
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) {
      const float* X = Xg + 4 * XF1 * tp;
      float vc[3][4];
#pragma unroll
      for (int ty = 0; ty < 3; ++ty)
#pragma unroll
        for (int ii = 0; ii < 4; ++ii)
          vc[ty][ii] = vt[((tp * 3 + ty) * kTileRows + 4 * ii + g) * (HP + 1) + ntd * 16 + n16];
#pragma unroll
      for (int ci = 0; ci < CPW; ++ci) {
        const int L = nh * (w + kF8Waves * ci) + h;
        if (L < NLT) {
          const int kc = L / NT;
          const int j = kc / DQ, qq = 4 * (kc % DQ) + (n16 >> 2);
#pragma unroll
          for (int ii = 0; ii < 4; ++ii) {
            const float xb = X[4 * ((j * QD + qq) * kTileRows + 4 * ii + g) + (n16 & 3)];
            if (j != C) {
              accW[ci] = mfma16x4(vc[0][ii], xb, accW[ci]);
            } else {
              const float xc = X[4 * ((WIN * QD + qq) * kTileRows + 4 * ii + g) + (n16 & 3)];
              accW[ci] = mfma16x4(vc[1][ii], xb, accW[ci]);
              accW[ci] = mfma16x4(vc[2][ii], xc, accW[ci]);
            }
          }
        }
      }
    }

    // ---- G: output tiles ot = nh (w + 16u) + h of the group (tile
    // ot / NGT, position j = (ot % NGT) / DQ, columns cb*16).
    // A operand: lane (r = n16, g) holds V_ty[r][4q + g]; B operand: lane
    // (col = n16, g) holds W1[4q + g][jj*D + cb*16 + col].
#pragma unroll
    for (int u = 0; u < GPW; ++u) {
      const int ot = nh * (w + kF8Waves * u) + h;
      if (ot < TP * NGT) {
        const int tp = ot / NGT, o = ot - tp * NGT;
        const int j = o / DQ, cb = o - (o / DQ) * DQ;
        const int ty = (j == WIN) ? 2 : (j == C ? 1 : 0);
        const int jj = (j == WIN) ? C : j;
        f4 acc = kZero4;
#pragma unroll
        for (int q = 0; q < HP / 4; ++q) {
          const float av = vt[((tp * 3 + ty) * kTileRows + n16) * (HP + 1) + 4 * q + g];
          const float bv = w1s[(4 * q + g) * S + jj * D + cb * 16 + n16];
          acc = mfma16x4(av, bv, acc);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = row0 + tp * kTileRows + 4 * g + i;
          if (row < a.B) __builtin_nontemporal_store(acc[i], &a.G[((size_t)row * W1P + j) * D + cb * 16 + n16]);
        }
      }
    }
  };

  if constexpr (TP == 1) {
    store_x(xr);
    __syncthreads();  // X (and W1) staged
    forward(xl);
    __syncthreads();  // forward partials written
    epilogue(tile0 * kTileRows);
    __syncthreads();  // V written
    backward(xl, tile0 * kTileRows);
  } else {
    // Pairs of tiles, four barriers per pair (X staged, forward partials, V,
    // and the end of the pair's dW1 before the next pair's rows overwrite
    // X).  tiles_per_wg is even, so the second tile of a pair is this
    // workgroup's, or past the last tile (rows >= B).
    // The next pair's ids take one set of registers: their rows are addressed
    // before the ids of the pair after it replace them.  (Two sets indexed by the
    // loop's counter came out of the compiler with one condition for both
    // writes: an odd gi wrote neither, and every second pair from the fourth on
    // read row 0.)
    const int ng = (ntl + 1) / 2;
    for (int gi = 0; gi < ng; ++gi) {
      const int row0 = (tile0 + 2 * gi) * kTileRows;
      store_x(xr);
      __syncthreads();  // X of this pair (and W1) staged
      if (gi + 1 < ng) {
        load_x(idn, xr);                                         // rows of the next pair
        if (gi + 2 < ng) load_ids(tile0 + 2 * (gi + 2), idn);    // ids two pairs ahead
      }
      forward(xl);
      __syncthreads();  // forward partials written
      epilogue(row0);
      __syncthreads();  // V written
      backward(xl, row0);
      if (gi + 1 < ng) __syncthreads();  // X and vt free (uniform branch)
    }
  }

  // ---- this workgroup's partial of the dense gradients (streaming stores,
  // like the G rows above: the next kernel reads them once).  Slot layout:
  // dW1 [Hp][K], db1 [Hp], dw2 [Hp], loss, db2.
  float* P = a.part + (size_t)wg * a.part_stride;
#pragma unroll
  for (int ci = 0; ci < CPW; ++ci) {
    const int L = nh * (w + kF8Waves * ci) + h;
    if (L < NLT) {
      const int kc = L / NT;
#pragma unroll
      for (int i = 0; i < 4; ++i) __builtin_nontemporal_store(accW[ci][i], &P[(ntd * 16 + 4 * g + i) * K + kc * 16 + n16]);
    }
  }
  // db1, dw2 (per hidden unit: the two row halves of the wave, then the
  // waves in order), loss (one value per wave); db2 is identically 0 (both
  // scores share b2)
  db1a += __shfl_xor(db1a, 32);
  dw2a += __shfl_xor(dw2a, 32);
  for (int o = 1; o < kWave; o <<= 1) lossa += __shfl_xor(lossa, o);
  float* rw = red + w * (2 * HP + 2);
  if (rsel == 0 && hn < HP) {
    rw[hn] = db1a;
    rw[HP + hn] = dw2a;
  }
  if (lane == 0) {
    rw[2 * HP] = lossa;
    rw[2 * HP + 1] = 0.f;
  }
  __syncthreads();
  if (w == 0 && h == 0) {
    for (int e = lane; e < 2 * HP + 2; e += kWave) {
      float s = red[e];
#pragma unroll
      for (int v = 1; v < kF8Waves; ++v) s += red[v * (2 * HP + 2) + e];
      P[HP * K + e] = s;
    }
  }
}

}  // namespace pg
