// The fused step kernel for d 64, window 5, 17 <= H <= 32 at batches whose
// sort runs elsewhere: gather + forward + hinge + backward of 32-window tiles
// on the bfloat16 matrix instructions (16x16x32), every float32 operand split
// exactly into three bfloat16 terms (lg_split8), ending in the per-entry rows
// G and this workgroup's dense partials like the other forms.
//
// One workgroup of 8 waves per CU.  A 32-window tile is one contraction step
// of dW1, and the 32 hidden units one step of G.  W1 stays in registers: each
// wave holds the fragments of its share of the forward (hidden block w & 1,
// three of the twelve column steps) and of its three G blocks, 72 registers.
// A tile's embedding rows are split once and sit in LDS as forward operands
// [column step][row tile][term][16 lanes of rows x 4 of columns][8 columns];
// dW1 needs eight windows of one column per lane and reads the same words
// through the transposing LDS read.  V = dz + dz~, dz, dz~ is written once, in
// the order the epilogue's lanes hold it (a dW1 operand: eight windows of one
// hidden unit), and G reads it transposed.
//
// Phases of a tile, a barrier after each:
//   F  forward: partial sums over the column steps (the centre block's true
//      and corrupted sums apart: z = zc + zctr, z~ = zc + zcor, §1 model, x~)
//   E  epilogue: wave (row tile w & 1, row w >> 1 of each group of four)
//   B  dW1 (a tile's first products and the rest apart, as everywhere; their
//      sum joins the registers' total of the tiles) and G; the next tile's
//      rows, in flight since F, are split after the matrix instructions
//   S  the split rows go to LDS
// Timestamps at B = 65,536 (8 tiles per workgroup, cycles at about 2.1 GHz; before
// the terms were rounded to nearest and a tile's sums kept apart, which cost 2.3
// of 53.8 us per launch): W1
// and the first rows 10,400, then per tile F 4,300, E 2,200, B 5,500, S 1,100.
// The 108 matrix instructions of a wave take 3,460 of them on a SIMD of two
// waves (counters: 19% of a launch): the rest is vector-ALU work (splits, tanh, sums, addresses) that the
// barriers keep from running under them.  Against the float32 form it replaced
// (12 waves in roles, 42% of the cycles in matrix instructions at 4 times the
// number): 71 -> 56 us per launch at B = 65,536, 29 -> 22 us at 16,384.  The
// gradients' error against 64 bits (norm of the difference over the norm, six
// batches of 65,536): rows of E 5.6e-8 -> 5.5e-8, W1 6.5e-8 -> 5.7e-8, b1 1.9e-7
// -> 1.0e-7, w2 1.2e-7 -> 6.9e-8; of 4,096: 5.8e-8 -> 5.2e-8, 6.4e-8 -> 5.5e-8,
// 1.7e-7 -> 1.2e-7, 9.7e-8 -> 7.6e-8.
#pragma once
#include "common.h"
#include "large_dev.h"
#include "launch.h"

namespace pg {

typedef short fs4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) fs4 fs4_lds;

struct FsShape {
  static constexpr int D = 64, WIN = 5, C = 2, W1P = 6, K = 320, HP = 32;
  static constexpr int R = kFsRows;                          // windows per tile
  static constexpr int X = 2 * W1P * 2 * 3 * kWave;          // 16-byte words of a tile's rows
  static constexpr int V = 3 * 2 * 3 * kWave;                // ... of its vectors
  static constexpr int Z = 4 * 2 * 2 * 4 * kWave;            // floats of the zc partials, and of
                                                             // the zctr and zcor ones
  static constexpr int kLds = (X + V) * 16 + 2 * Z * 4 + 2 * R * W1P * 4 + 8 * (2 * HP + 2) * 4;
  static_assert(kLds <= kMaxLdsBytes, "LDS of one workgroup");
};

typedef uint32_t lu2 __attribute__((ext_vector_type(2)));
// Eight 16-bit terms: four rows of each of two 8-byte-word arrays, transposed
// inside groups of 16 lanes (lane 4 r + q gives columns 4q.. of row r and gets
// column 4 r + q of the four rows).
__device__ __forceinline__ lu4 fs_read_tr(const lu2* p0, const lu2* p1) {
  const lu2 x = __builtin_bit_cast(lu2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((fs4_lds*)p0));
  const lu2 y = __builtin_bit_cast(lu2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((fs4_lds*)p1));
  return lu4{x[0], x[1], y[0], y[1]};
}

// Sum over the 16 lanes of a row, in every lane.
template <int CTRL>
__device__ __forceinline__ float fs_ror(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float fs_row_sum(float x) {
  return fs_ror<0x121>(fs_ror<0x122>(fs_ror<0x124>(fs_ror<0x128>(x))));
}

__device__ inline void fwdbwd_split(const FwdArgs& a, int wg, char* lds) {
  using Sh = FsShape;
  constexpr int D = Sh::D, C = Sh::C, W1P = Sh::W1P, K = Sh::K, HP = Sh::HP, R = Sh::R;
  constexpr int NT = kFsThreads;
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int i = lane & 15, g = lane >> 4;
  lu4* xs = reinterpret_cast<lu4*>(lds);
  lu2* vs = reinterpret_cast<lu2*>(xs + Sh::X);  // [type][n][term][m][64] 8-byte words
  float* zc = reinterpret_cast<float*>(xs + Sh::X + Sh::V);  // [4 shares][m][n][4][64]
  float* zd = zc + Sh::Z;                            // [2 shares][ctr, cor][m][n][4][64]
  int32_t* idt = reinterpret_cast<int32_t*>(zd + Sh::Z);  // [2][R][W1P]
  float* red = reinterpret_cast<float*>(idt + 2 * R * W1P);  // [8][2 HP + 2]
  const int tile0 = wg * a.tiles_per_wg;
  const int ntl = min(a.tiles_per_wg, a.ntiles - tile0);  // tiles of this workgroup (>= 1)

  // ids of a tile: thread t < 192 takes entry t (row t / 6, position t % 6)
  auto load_id = [&](int tile) LG_INLINE {
    const int r = t / W1P, j = t - r * W1P, b = tile * R + r;
    int32_t id = 0;
    if (t < R * W1P && b < a.B) id = j < Sh::WIN ? a.windows[(size_t)b * Sh::WIN + j] : a.corrupt[b];
    return id;
  };
  auto store_id = [&](int buf, int32_t id) LG_INLINE {  // (rows >= B and bad ids read row 0)
    const bool bad = (uint32_t)id >= (uint32_t)a.V;
    if (bad) atomicOr(a.flag, kFlagBadId);
    if (t < R * W1P) idt[buf * R * W1P + t] = bad ? 0 : id;
  };
  // unit u = t + 512 v of a tile's rows: row 16 (u / 64 % 2) + u % 16, column
  // step u / 128 (position u / 256), columns 8 (u / 16 % 4) of it
  f4 xr[3][2];
  auto load_x = [&](int buf) LG_INLINE {
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      const int u = t + v * NT, ks = u >> 7;
      const int r = 16 * ((u >> 6) & 1) + (u & 15), col = 32 * (ks & 1) + 8 * ((u >> 4) & 3);
      const float* src = a.E + (size_t)idt[buf * R * W1P + r * W1P + (ks >> 1)] * D + col;
      xr[v][0] = ld4(src);
      xr[v][1] = ld4(src + 4);
    }
  };
  lu4 xp[3][3];
  auto split_x = [&](int tile) LG_INLINE {
    float x[3][8], big = 0.f;
    if ((tile + 1) * R > a.B)  // rows past the batch are zero (a NaN of row 0 would reach dW1)
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        const int u = t + v * NT;
        if (tile * R + 16 * ((u >> 6) & 1) + (u & 15) >= a.B) xr[v][0] = xr[v][1] = kZero4;
      }
#pragma unroll
    for (int v = 0; v < 3; ++v) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[v][e] = xr[v][e >> 2][e & 3];
      lg_largest(x[v], big);
    }
    lg_checked(big, [&](auto safe) LG_INLINE {
#pragma unroll
      for (int v = 0; v < 3; ++v) lg_split8<decltype(safe)::value>(x[v], xp[v]);
    });
  };
  auto store_x = [&]() LG_INLINE {
#pragma unroll
    for (int v = 0; v < 3; ++v)
#pragma unroll
      for (int k = 0; k < 3; ++k) xs[(((t + v * NT) >> 6) * 3 + k) * kWave + lane] = xp[v][k];
  };

  int32_t idn = load_id(tile0);
  store_id(0, idn);
  __syncthreads();
  load_x(0);  // in flight while W1 is loaded and split
  idn = ntl > 1 ? load_id(tile0 + 1) : 0;
  // the forward's share: hidden block n = w & 1, share kq = w >> 1 of the
  // units (column step of X, column step of W1): 0 1 2 | 3, 4, corrupt 0 |
  // 6, 5, corrupt 1 | 7 8 9
  const int nf = w & 1, kq = w >> 1;
  const bool mid = kq == 1 || kq == 2;
  const int xu[3] = {kq == 0 ? 0 : (kq == 1 ? 3 : (kq == 2 ? 6 : 7)),
                     kq == 0 ? 1 : (kq == 1 ? 4 : (kq == 2 ? 5 : 8)),
                     kq == 0 ? 2 : (kq == 1 ? 10 : (kq == 2 ? 11 : 9))};
  float wx[6][8], wbig = 0.f;  // the forward's three units, then G's three blocks
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int ks = xu[u] >= 2 * Sh::WIN ? xu[u] - 2 * (Sh::WIN - C) : xu[u];
    const int n = 16 * nf + i;
    const float* src = a.W1 + (size_t)(n < a.H ? n : 0) * K + 32 * ks + 8 * g;
    const f4 v0 = ld4(src), v1 = ld4(src + 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) wx[u][e] = n < a.H ? (e < 4 ? v0[e & 3] : v1[e & 3]) : 0.f;
    lg_largest(wx[u], wbig);
  }
  // the backward's blocks: block 3w + u of the 24 (position pu, 16 columns at
  // 16 cq) ordered true centre, corrupt, contexts, so that most waves need one
  // type of vector
  int pu[3], cq[3], ty[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int L = 3 * w + u, o = L >> 2;
    cq[u] = L & 3;
    pu[u] = o == 0 ? C : (o == 1 ? Sh::WIN : (o < 4 ? o - 2 : o - 1));
    ty[u] = o == 0 ? 1 : (o == 1 ? 2 : 0);
  }
  lu4 wf[3][3], wg3[3][3];  // wg3, lane (i, g): W1[4g .. 4g + 3 and 16 + 4g ..][column i]
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int blk = pu[u] == Sh::WIN ? C : pu[u];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int h = 16 * (e >> 2) + 4 * g + (e & 3);
      const float x = a.W1[(size_t)(h < a.H ? h : 0) * K + blk * D + 16 * cq[u] + i];
      wx[3 + u][e] = h < a.H ? x : 0.f;
    }
    lg_largest(wx[3 + u], wbig);
  }
  lg_checked(wbig, [&](auto safe) LG_INLINE {
#pragma unroll
    for (int u = 0; u < 3; ++u) lg_split8<decltype(safe)::value>(wx[u], wf[u]);
#pragma unroll
    for (int u = 0; u < 3; ++u) lg_split8<decltype(safe)::value>(wx[3 + u], wg3[u]);
  });
  float b1v[2], w2v[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int h = 16 * n + i;
    b1v[n] = h < a.H ? a.b1[h] : 0.f;
    w2v[n] = h < a.H ? a.w2[h] : 0.f;
  }
  const float b2v = a.b2[0];
  split_x(tile0);
  store_x();
  store_id(1, idn);
  __syncthreads();

  f4 accW[3][2];
#pragma unroll
  for (int u = 0; u < 3; ++u) accW[u][0] = accW[u][1] = kZero4;
  float db1a[2] = {0.f, 0.f}, dw2a[2] = {0.f, 0.f}, lossa = 0.f;
  constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};

  for (int tt = 0; tt < ntl; ++tt) {
    // the lane's coordinates anew for each tile, so that no address is kept in
    // registers across the phases
    int lane_o = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane_o));
    const int lane = lane_o, i = lane & 15, g = lane >> 4;
    const int row0 = (tile0 + tt) * R;
    const bool more = tt + 1 < ntl;
    if (more) load_x((tt + 1) & 1);
    idn = tt + 2 < ntl ? load_id(tile0 + tt + 2) : 0;

    // ---- F
    {
      f4 s[3][2];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        lu4 A[2][3];
        lg_read<2>(xs + xu[u] * 2 * 3 * kWave + lane, A);
        f4 hi[2] = {kZero4, kZero4}, lo[2] = {kZero4, kZero4};
#pragma unroll
        for (int p = 0; p < 5; ++p)
#pragma unroll
          for (int m = 0; m < 2; ++m) lo[m] = lg_mfma(A[m][PA[p]], wf[u][PB[p]], lo[m]);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          hi[m] = lg_mfma(A[m][0], wf[u][0], hi[m]);
          s[u][m] = lg_sum(hi[m], lo[m]);
        }
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const f4 z = mid ? s[0][m] : (s[0][m] + s[1][m]) + s[2][m];
        float* dst = zc + ((kq * 2 + m) * 2 + nf) * 4 * kWave + lane;
#pragma unroll
        for (int c = 0; c < 4; ++c) dst[c * kWave] = z[c];
        if (mid) {
          float* d1 = zd + ((((kq - 1) * 2 + 0) * 2 + m) * 2 + nf) * 4 * kWave + lane;
          float* d2 = zd + ((((kq - 1) * 2 + 1) * 2 + m) * 2 + nf) * 4 * kWave + lane;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            d1[c * kWave] = s[1][m][c];
            d2[c * kWave] = s[2][m][c];
          }
        }
      }
    }
    __syncthreads();

    // ---- E: lane (i, g) takes row 16m + 4g + q, hidden units i and 16 + i
    {
      const int m = w & 1, q = w >> 1, row = row0 + 16 * m + 4 * g + q;
      float h[2], ht[2], hmh[2], ps = 0.f, pst = 0.f;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        float Zc = 0.f, Zctr = 0.f, Zcor = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) Zc += zc[(((k * 2 + m) * 2 + n) * 4 + q) * kWave + lane];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          Zctr += zd[((((k * 2 + 0) * 2 + m) * 2 + n) * 4 + q) * kWave + lane];
          Zcor += zd[((((k * 2 + 1) * 2 + m) * 2 + n) * 4 + q) * kWave + lane];
        }
        h[n] = tanh_fast(b1v[n] + (Zc + Zctr));
        ht[n] = tanh_fast(b1v[n] + (Zc + Zcor));
        // h - h~ = tanh(z - z~) (1 - h h~)
        hmh[n] = tanh_fast(Zctr - Zcor) * (1.f - h[n] * ht[n]);
        ps += w2v[n] * h[n];
        pst += w2v[n] * ht[n];
      }
      ps = fs_row_sum(ps);
      pst = fs_row_sum(pst);
      const float mg = 1.f - (b2v + ps) + (b2v + pst);
      const bool live = row < a.B;           // rows past the batch add nothing, whatever they hold
      const bool on = live && mg > 0.f;       // hinge active (derivative 0 at margin 0)
      const float gst = on ? a.invB : 0.f;    // d loss/d s~ = m/B, d loss/d s = -m/B
      uint16_t* vt = reinterpret_cast<uint16_t*>(vs) + (m * kWave + lane) * 4 + q;
      float v[2][3], big = 0.f;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const float gw = gst * w2v[n];
        v[n][0] = live ? gw * hmh[n] * (h[n] + ht[n]) : 0.f;
        v[n][1] = live ? -gw * (1.f - h[n] * h[n]) : 0.f;
        v[n][2] = live ? gw * (1.f - ht[n] * ht[n]) : 0.f;
        lg_largest(v[n], big);
        db1a[n] += v[n][0];
        dw2a[n] -= live ? gst * hmh[n] : 0.f;  // -(m/B) h + (m/B) h~
      }
      lg_checked(big, [&](auto safe) LG_INLINE {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int y = 0; y < 3; ++y) {
            const uint32_t u = lg_first2<decltype(safe)::value>(v[n][y], v[n][y]);
            const float r = v[n][y] - __uint_as_float(u << 16);
            const uint32_t mm = lg_round2(r, r);
            const float q3 = r - __uint_as_float(mm << 16);
            uint16_t* d = vt + (y * 2 + n) * 3 * 2 * kWave * 4;
            d[0] = (uint16_t)u;
            d[2 * kWave * 4] = (uint16_t)mm;
            d[2 * 2 * kWave * 4] = (uint16_t)(__float_as_uint(q3) >> 16);
          }
      });
      if (i == 0) lossa += on ? mg : 0.f;
    }
    store_id(tt & 1, idn);
    __syncthreads();

    // ---- B
    {
      const int r4 = (lane & 15) >> 2, c4 = lane & 3;
      const int row = 4 * g + r4;  // the transposing reads: rows 4g .. of a group of 16 lanes
      lu4 A[2][3];
      // dW1: V^T (hidden tiles n) times the rows' 16 columns
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        if (u == 0 || ty[u] != ty[u - 1]) {
          const lu2* vb = vs + ty[u] * 2 * 3 * 2 * kWave + lane;
#pragma unroll
          for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int p = 0; p < 3; ++p) {
              const lu2 x = vb[(n * 3 + p) * 2 * kWave], y = vb[((n * 3 + p) * 2 + 1) * kWave];
              A[n][p] = lu4{x[0], x[1], y[0], y[1]};
            }
        }
        lu4 Bv[3];
        const lu2* x0 = reinterpret_cast<const lu2*>(
                            xs + ((2 * pu[u] + (cq[u] >> 1)) * 2) * 3 * kWave +
                            16 * (2 * (cq[u] & 1) + (c4 >> 1)) + row) + (c4 & 1);
#pragma unroll
        for (int p = 0; p < 3; ++p)
          Bv[p] = fs_read_tr(x0 + 2 * p * kWave, x0 + 2 * (3 + p) * kWave);
        f4 hi[2] = {kZero4, kZero4}, lo[2] = {kZero4, kZero4};
#pragma unroll
        for (int p = 0; p < 5; ++p)
#pragma unroll
          for (int n = 0; n < 2; ++n) lo[n] = lg_mfma(A[n][PA[p]], Bv[PB[p]], lo[n]);
#pragma unroll
        for (int n = 0; n < 2; ++n) hi[n] = lg_mfma(A[n][0], Bv[0], hi[n]);
#pragma unroll
        for (int n = 0; n < 2; ++n) accW[u][n] += lg_sum(hi[n], lo[n]);
        // (keeps the sums out of the compiler's reach: it spills 24 to 69 registers
        // over the loop without this)
        asm volatile("" : "+v"(accW[u][0]), "+v"(accW[u][1]));
      }
      lg_pin();
      // G: V (row tiles m) times W1's 16 columns
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        if (u == 0 || ty[u] != ty[u - 1]) {
          const lu2* vb = vs + ty[u] * 2 * 3 * 2 * kWave + 16 * c4 + row;
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int p = 0; p < 3; ++p)
              A[m][p] = fs_read_tr(vb + (p * 2 + m) * kWave, vb + ((3 + p) * 2 + m) * kWave);
        }
        f4 hi[2] = {kZero4, kZero4}, lo[2] = {kZero4, kZero4};
#pragma unroll
        for (int p = 0; p < 5; ++p)
#pragma unroll
          for (int m = 0; m < 2; ++m) lo[m] = lg_mfma(A[m][PA[p]], wg3[u][PB[p]], lo[m]);
#pragma unroll
        for (int m = 0; m < 2; ++m) hi[m] = lg_mfma(A[m][0], wg3[u][0], hi[m]);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const f4 v = lg_sum(hi[m], lo[m]);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int b = row0 + 16 * m + 4 * g + c;
            if (b < a.B)
              __builtin_nontemporal_store(v[c], &a.G[((size_t)b * W1P + pu[u]) * D + 16 * cq[u] + i]);
          }
        }
      }
    }
    if (more) split_x(tile0 + tt + 1);
    __syncthreads();

    // ---- S
    if (more) {
      store_x();
      __syncthreads();
    }
  }

  // ---- this workgroup's partial: dW1 [HP][K], db1 [HP], dw2 [HP], loss, db2
  float* P = a.part + (size_t)wg * a.part_stride;
  // the centre block's corrupt half (blocks 4-7) joins its true one (0-3)
  f4* cx = reinterpret_cast<f4*>(xs);  // [cq][n][64]; the rows are done with
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (pu[u] == Sh::WIN)
#pragma unroll
      for (int n = 0; n < 2; ++n) cx[(cq[u] * 2 + n) * kWave + lane] = accW[u][n];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (pu[u] != Sh::WIN)
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        f4 v = accW[u][n];
        if (pu[u] == C) v += cx[(cq[u] * 2 + n) * kWave + lane];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          P[(size_t)(16 * n + 4 * g + c) * K + pu[u] * D + 16 * cq[u] + i] = v[c];
      }
  float* rw = red + w * (2 * HP + 2);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    float x = db1a[n], y = dw2a[n];
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    if (g == 0) {
      rw[16 * n + i] = x;
      rw[HP + 16 * n + i] = y;
    }
  }
  for (int o = 1; o < kWave; o <<= 1) lossa += __shfl_xor(lossa, o);
  if (lane == 0) {
    rw[2 * HP] = lossa;
    rw[2 * HP + 1] = 0.f;  // both scores share b2: its gradient is 0
  }
  __syncthreads();
  for (int e = t; e < 2 * HP + 2; e += NT) {
    float s = red[e];
#pragma unroll
    for (int v = 1; v < 8; ++v) s += red[v * (2 * HP + 2) + e];
    P[(size_t)HP * K + e] = s;
  }
}

}  // namespace pg
