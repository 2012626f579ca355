// The SGD step for models whose W1 does not fit in a workgroup's LDS (hidden
// layer wider than 64 units, e.g. d 128, window 11, H 256): three contractions
// on the bfloat16 matrix instructions, each float32 operand split exactly
// into three bfloat16 terms, with the embedding rows gathered on the fly.
//
//   k_large_prep  W1 split and laid out as MFMA operand fragments, once for
//                 the forward (contraction over the window's columns) and once
//                 for the rows G (contraction over the hidden units).
//   k_large_fwd   Z = X W1^T and, for the corrupted copy, the centre-block
//                 difference D = (e~ - e_c) W1_c^T (so z~ = z + D; §1 model,
//                 x~); then tanh, both scores, hinge and the per-window
//                 vectors V = (dz + dz~, dz, dz~), written to global memory,
//                 and this workgroup's db1 / dw2 / loss partial.  In score-only
//                 form it writes s(x) instead.
//   k_large_dw1   dW1 partials: dW1[h][k] = sum_b V_b[h] x_b[k] over slices of
//                 the batch (centre block: dz e_c, and in columns of its own
//                 dz~ e~).
//   k_large_g     G[e][:] = W1_j^T V for entry e = b(win+1) + j (context
//                 positions dz + dz~, the true centre dz, the corrupt entry dz~
//                 through block c).
// Rows b >= B read row 0 (or zero) and are masked out of every result.
//
// The split.  x = x1 + x2 + x3, each term what is left rounded to 8 significant
// bits; the three hold all 24.  Rounding to nearest keeps x2 within 2^-8 of x's
// leading bit and x3 within 2^-17, and without a preferred sign.  Of the nine
// products six are kept; the others (x2 y3, x3 y2, x3 y3) are below 2^-24 of the
// product, a float32 rounding, and 2^-27.4 in the root mean square (normal
// operands; truncating x1 instead left 2^-22.0 and 2^-25.4, the former with one
// sign where entries repeat).  An operand below 2^-110 keeps what lies above
// 2^-133, the smallest bfloat16.  x1 y1 goes to an accumulator of its own and the
// other five to a second one, so a contraction rounds at the size of its sum once
// per 32 terms, where the float32 instruction rounds once per 4: the largest error
// of 256 random terms over the sum of their magnitudes is 0.8 x 2^-24, that of the
// float32 instruction 3.6 x 2^-24; of 256 equal ones 1.3 and 2.6.
// An infinite operand has finite companions no more (inf - inf), which only the
// second accumulator sees: a non-finite first sum is the result, as one float32
// chain would give it.
// Six bfloat16 products take 96 matrix cycles per 16x16x32 block, eight
// float32 ones 256.  Gradients of the d 128, window 11, H 256 model at B =
// 16,384, error against 64 bits (norm of the difference over the norm, six
// batches), float32 instructions -> this: rows of E 7.6e-8 -> 6.1e-8, W1 2.6e-7
// -> 5.9e-8, b1 3.4e-7 -> 1.6e-7, w2 8.3e-8 -> 6.2e-8.
#pragma once
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace pg {

// On the kernels' lambdas: one that is called from several places and not
// inlined takes the arrays it captures to scratch memory.
#define LG_INLINE __attribute__((always_inline))

typedef __bf16 lb8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f4 lg_mfma(lu4 a, lu4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lb8, a),
                                                 __builtin_bit_cast(lb8, b), c, 0, 0, 0);
}

// Two floats rounded to bfloat16 (to nearest), packed in order.
__device__ __forceinline__ uint32_t lg_round2(float x, float y) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x, y}, b2));
}

// Finite floats above the largest bfloat16 round to an infinity; as first terms
// they are truncated to it (the second term holds the rest).  Callers look for
// them once for all that a phase splits, and take its SAFE copy if one is there.
constexpr float kLgMax = 0x1.fep127f;
template <int N>
__device__ __forceinline__ void lg_largest(const float (&x)[N], float& big) {
#pragma unroll
  for (int e = 0; e < N; ++e) big = __builtin_elementwise_maximum(big, __builtin_fabsf(x[e]));
}
// f(std::true_type) if a lane of the wave has such a value (or an infinity, or a
// NaN, which would hide one), else f(std::false_type).
template <class F>
__device__ __forceinline__ void lg_checked(float big, F f) {
  if (__builtin_expect(__ballot(!(big <= kLgMax)) != 0, 0)) f(std::true_type{});
  else f(std::false_type{});
}
template <bool SAFE>
__device__ __forceinline__ uint32_t lg_first2(float x, float y) {
  if (SAFE && __builtin_fabsf(x) < __builtin_inff()) x = __builtin_amdgcn_fmed3f(x, -kLgMax, kLgMax);
  if (SAFE && __builtin_fabsf(y) < __builtin_inff()) y = __builtin_amdgcn_fmed3f(y, -kLgMax, kLgMax);
  return lg_round2(x, y);
}

// The three bfloat16 terms of eight floats, packed in order.
template <bool SAFE>
__device__ __forceinline__ void lg_split8(const float (&x)[8], lu4 (&p)[3]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const uint32_t u = lg_first2<SAFE>(x[2 * v], x[2 * v + 1]);
    p[0][v] = u;
    float r0 = x[2 * v] - __uint_as_float(u << 16);
    float r1 = x[2 * v + 1] - __uint_as_float(u & 0xffff0000u);
    const uint32_t m = lg_round2(r0, r1);
    p[1][v] = m;
    r0 -= __uint_as_float(m << 16);
    r1 -= __uint_as_float(m & 0xffff0000u);
    p[2][v] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
  }
}

// hi + lo, or hi alone where it is not finite.
__device__ __forceinline__ f4 lg_sum(f4 hi, f4 lo) {
  f4 r;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    r[q] = __builtin_fabsf(hi[q]) < __builtin_inff() ? hi[q] + lo[q] : hi[q];
  return r;
}

// A group of a 32-term step: P row tiles x 2 column tiles, hi/lo[m][n] +=
// A_m B[n], product-major (dependent instructions on one accumulator issue
// back to back at full rate).
template <int P>
__device__ __forceinline__ void lg_read(const lu4* s, lu4 (&A)[P][3]) {
#pragma unroll
  for (int v = 0; v < P; ++v)
#pragma unroll
    for (int k = 0; k < 3; ++k) A[v][k] = s[(v * 3 + k) * kWave];
}
template <int P, int MT>
__device__ __forceinline__ void lg_group(const lu4 (&A)[P][3], const lu4 (&Bv)[2][3], int m0,
                                         f4 (&hi)[MT][2], f4 (&lo)[MT][2]) {
  constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
  for (int p = 0; p < 5; ++p)
#pragma unroll
    for (int v = 0; v < P; ++v)
#pragma unroll
      for (int n = 0; n < 2; ++n)
        lo[m0 + v][n] = lg_mfma(A[v][PA[p]], Bv[n][PB[p]], lo[m0 + v][n]);
#pragma unroll
  for (int v = 0; v < P; ++v)
#pragma unroll
    for (int n = 0; n < 2; ++n) hi[m0 + v][n] = lg_mfma(A[v][0], Bv[n][0], hi[m0 + v][n]);
}
// Keeps the reads issued above it ahead of the instructions below it.
__device__ __forceinline__ void lg_pin() { __builtin_amdgcn_sched_barrier(0); }

// One 32-term step of MT row tiles (fragments at s), row tiles in pairs.
template <int MT>
__device__ __forceinline__ void lg_step(const lu4* s, const lu4 (&Bv)[2][3], f4 (&hi)[MT][2],
                                        f4 (&lo)[MT][2]) {
  constexpr int P = MT > 1 ? 2 : 1;
#pragma unroll
  for (int m = 0; m < MT; m += P) {
    lu4 A[P][3];
    lg_read<P>(s + m * 3 * kWave, A);
    lg_group<P, MT>(A, Bv, m, hi, lo);
  }
}

// =============================================================== W1 fragments
//
// A fragment is one operand of one MFMA: 64 lanes x 8 bfloat16 (16 bytes a
// lane), lane (i, g) holding terms 8g..8g+7 of row i.
//   wf[K/32 step][H/16 block][3 terms][64]  W1[16 hb + i][32 ks + 8g ..]
//   wg[K/16 block][H/32 step][3 terms][64]  W1[32 hs + 8g ..][16 cb + i]
// One wave per fragment triple; both layouts in one launch (the fragments of
// wg follow those of wf).  4 us for H 256 x K 1408; without it every forward
// and G workgroup would split W1 again (360,448 values, 256 times).
__global__ __launch_bounds__(kBlock) void k_large_prep(LargeArgs a) {
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int i = lane & 15, g = lane >> 4;
  const int n = a.H * a.K / 512;  // fragments of one layout
  int u = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + t / kWave);
  if (u >= 2 * n) return;
  float x[8];
  lu4* dst;
  if (u < n) {
    const int hb = u % (a.H / 16), ks = u / (a.H / 16);
    const float* src = a.W1 + (size_t)(16 * hb + i) * a.K + 32 * ks + 8 * g;
    const f4 v0 = ld4(src), v1 = ld4(src + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[e] = v0[e];
      x[4 + e] = v1[e];
    }
    dst = a.wf + (size_t)u * 3 * kWave;
  } else {
    u -= n;
    const int hs = u % (a.H / 32), cb = u / (a.H / 32);
    const float* src = a.W1 + (size_t)(32 * hs + 8 * g) * a.K + 16 * cb + i;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = src[(size_t)e * a.K];
    dst = a.wg + (size_t)u * 3 * kWave;
  }
  float big = 0.f;
  lg_largest(x, big);
  lg_checked(big, [&](auto safe) LG_INLINE {
    lu4 p[3];
    lg_split8<decltype(safe)::value>(x, p);
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[k * kWave + lane] = p[k];
  });
}

// =============================================================== forward
//
// NW = H / 32 waves, wave w owning hidden units [32w, 32w + 32) of the
// workgroup's 16 MT windows.  The windows' rows go through LDS in chunks of 64
// columns as A fragments, double-buffered, the next chunk's rows in flight
// in registers; W1's fragments belong to one wave each and come
// straight from memory (the L2: every workgroup walks them in the same order),
// one step ahead.  The centre block comes first, so that D's second
// accumulator is gone before the other chunks.  Bound: the matrix
// instructions, and for few windows the 6 H K bytes of fragments that every
// workgroup reads, hence the smallest MT that needs at most one workgroup per
// CU (large_fwd_mt).
template <int NW, int MT, bool SCORE>
__global__ __launch_bounds__(NW * kWave) void k_large_fwd(LargeArgs a) {
  constexpr int R = 16 * MT, NT = NW * kWave;
  constexpr int UN = R * 8;                    // 8-column units of a chunk
  constexpr int UPT = (UN + NT - 1) / NT;      // ... per thread
  constexpr int SF = MT * 3 * kWave;           // fragment words of one step
  __shared__ lu4 Xs[2][2 * SF];
  __shared__ lu4 Ts[SCORE ? 1 : 2][SCORE ? 1 : 2 * SF];
  __shared__ int32_t ids[R][kMaxWin + 1];
  __shared__ float sred[2][NW][R];
  __shared__ float gsh[R];
  __shared__ int badrow[R];
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int i = lane & 15, g = lane >> 4;
  const int r0 = blockIdx.x * R;
  // one wave of each SIMD goes first, so the two drift apart and one's reads
  // and epilogues run under the other's matrix instructions
  if (w >= NW / 2) __builtin_amdgcn_s_setprio(1);
  const int W1p = a.win + 1, d = a.d;
  if (t < R) badrow[t] = 0;
  __syncthreads();
  for (int k = t; k < R * W1p; k += NT) {
    const int r = k / W1p, j = k - r * W1p;
    const int b = r0 + r;
    int32_t id = 0;  // the score has no corrupt ids
    if (b < a.B && (j < a.win || !SCORE))
      id = j < a.win ? a.windows[(size_t)b * a.win + j] : a.corrupt[b];
    const bool bad = (uint32_t)id >= (uint32_t)a.V_rows;
    if (bad) {
      atomicOr(a.flag, kFlagBadId);
      badrow[r] = 1;
    }
    ids[r][j] = bad ? 0 : id;
  }
  __syncthreads();

  const int dch = d / 64, nch = a.K / 64, hb = a.H / 16;
  // chunk q in the order of work: the centre block's, then the others
  auto chunk_of = [&](int q) LG_INLINE {
    return q < dch ? a.c * dch + q : (q < (a.c + 1) * dch ? q - dch : q);
  };
  f4 X[UPT][2], C[UPT][2];
  // unit u of a chunk: row 16 (u / 128) + (u & 15), columns 32 ks + 8 g ..
  auto load = [&](int q) LG_INLINE {
    const int kc = chunk_of(q), jb = kc / dch, off = (kc - jb * dch) * 64;
#pragma unroll
    for (int v = 0; v < UPT; ++v) {
      const int u = t + v * NT;
      if (UN % NT == 0 || u < UN) {
        const int r = 16 * (u >> 7) + (u & 15), col = off + 32 * ((u >> 6) & 1) + 8 * ((u >> 4) & 3);
        const float* src = a.E + (size_t)ids[r][jb] * d + col;
        X[v][0] = ld4(src);
        X[v][1] = ld4(src + 4);
        if (!SCORE && q < dch) {
          const float* sc = a.E + (size_t)ids[r][a.win] * d + col;
          C[v][0] = ld4(sc);
          C[v][1] = ld4(sc + 4);
        }
      }
    }
  };
  auto store = [&](auto centre, int buf) LG_INLINE {
    constexpr bool CTR = decltype(centre)::value;
    float x[UPT][8], dx[UPT][8], big = 0.f;
#pragma unroll
    for (int v = 0; v < UPT; ++v) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[v][e] = X[v][e >> 2][e & 3];
        if (CTR) dx[v][e] = C[v][e >> 2][e & 3] - x[v][e];
      }
      if (UN % NT == 0 || t + v * NT < UN) {
        lg_largest(x[v], big);
        if (CTR) lg_largest(dx[v], big);
      }
    }
    lg_checked(big, [&](auto safe) LG_INLINE {
      constexpr bool SAFE = decltype(safe)::value;
#pragma unroll
      for (int v = 0; v < UPT; ++v) {
        const int u = t + v * NT;
        if (UN % NT == 0 || u < UN) {
          const int slot = (((u >> 6) & 1) * MT + (u >> 7)) * 3 * kWave + (u & 63);
          lu4 p[3];
          lg_split8<SAFE>(x[v], p);
#pragma unroll
          for (int k = 0; k < 3; ++k) Xs[buf][slot + k * kWave] = p[k];
          if constexpr (CTR) {
            lg_split8<SAFE>(dx[v], p);
#pragma unroll
            for (int k = 0; k < 3; ++k) Ts[buf][slot + k * kWave] = p[k];
          }
        }
      }
    });
  };
  auto load_w = [&](int q, int ks, lu4 (&Bv)[2][3]) LG_INLINE {
    const lu4* src = a.wf + ((size_t)(2 * chunk_of(q) + ks) * hb + 2 * w) * 3 * kWave + lane;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int k = 0; k < 3; ++k) Bv[n][k] = src[(n * 3 + k) * kWave];
  };
  f4 zh[MT][2], zl[MT][2], D[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) zh[m][n] = zl[m][n] = D[m][n] = kZero4;
  lu4 B0[2][3], B1[2][3];
  f4 dh[MT][2], dl[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) dh[m][n] = dl[m][n] = kZero4;
  // the next chunk's rows into the other buffer, the one after that into registers
  auto stage = [&](int q) LG_INLINE {
    if (q + 1 < nch) {
      if (!SCORE && q + 1 < dch) store(std::true_type{}, (q + 1) & 1);
      else store(std::false_type{}, (q + 1) & 1);
    }
    if (q + 2 < nch) load(q + 2);
  };
  load(0);
  load_w(0, 0, B0);
  load_w(0, 1, B1);
  store(std::integral_constant<bool, !SCORE>{}, 0);
  if (nch > 1) load(1);
  __syncthreads();
  // chunk q, in buffer q & 1: one barrier each.  The two waves of a SIMD stage
  // at opposite ends of the chunk, so that one splits while the other multiplies.
  auto chunk = [&](auto centre, int q) LG_INLINE {
    const int buf = q & 1;
    if (w < NW / 2) stage(q);
    const int qn = min(q + 1, nch - 1);  // (the last chunk's own again: not used)
    if constexpr (decltype(centre)::value) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        lu4 (&Bv)[2][3] = ks ? B1 : B0;
        lg_step<MT>(&Xs[buf][ks * SF + lane], Bv, zh, zl);
        lg_step<MT>(&Ts[buf][ks * SF + lane], Bv, dh, dl);
        load_w(qn, ks, Bv);
      }
    } else {
      constexpr int P = MT > 1 ? 2 : 1, GS = MT / P;  // groups of a step
      const lu4* s = &Xs[buf][lane];
      lu4 A[2][P][3];
      lg_read<P>(s, A[0]);
#pragma unroll
      for (int gr = 0; gr < 2 * GS; ++gr) {
        if (gr + 1 < 2 * GS) lg_read<P>(s + (gr + 1) * P * 3 * kWave, A[(gr + 1) & 1]);
        lg_pin();
        lg_group<P, MT>(A[gr & 1], gr / GS ? B1 : B0, gr % GS * P, zh, zl);
        lg_pin();
        if (gr % GS == GS - 1) load_w(qn, gr / GS, gr / GS ? B1 : B0);
      }
    }
    if (w >= NW / 2) stage(q);
    __syncthreads();
  };
  int q = 0;
  if constexpr (!SCORE) {
    for (; q < dch; ++q) chunk(std::true_type{}, q);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) D[m][n] = lg_sum(dh[m][n], dl[m][n]);
  }
  for (; q < nch; ++q) chunk(std::false_type{}, q);

  // ---- epilogue.  Lane (i, g), component q of Z[m][n]: row 16m + 4g + q,
  // hidden 32w + 16n + i.  Z becomes h, and ht holds h~.
  float b1v[2], w2v[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    b1v[n] = a.b1[32 * w + 16 * n + i];
    w2v[n] = a.w2[32 * w + 16 * n + i];
  }
  f4 ht[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    float s[4] = {0.f, 0.f, 0.f, 0.f}, st[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const f4 z = lg_sum(zh[m][n], zl[m][n]);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float zb = z[c] + b1v[n];
        zh[m][n][c] = tanh_fast(zb);
        s[c] += w2v[n] * zh[m][n][c];
        if (!SCORE) {
          ht[m][n][c] = tanh_fast(zb + D[m][n][c]);
          st[c] += w2v[n] * ht[m][n][c];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        s[c] += __shfl_xor(s[c], o);
        if (!SCORE) st[c] += __shfl_xor(st[c], o);
      }
      if (i == 0) {
        sred[0][w][16 * m + 4 * g + c] = s[c];
        if (!SCORE) sred[1][w][16 * m + 4 * g + c] = st[c];
      }
    }
  }
  __syncthreads();
  float lossr = 0.f;
  if (t < R) {
    float s = 0.f, st = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      s += sred[0][v][t];
      if (!SCORE) st += sred[1][v][t];
    }
    const int b = r0 + t;
    const float b2v = a.b2[0];
    if (SCORE) {
      if (b < a.B) a.scores[b] = badrow[t] ? __builtin_nanf("") : b2v + s;
    } else {
      const float mg = 1.f - (b2v + s) + (b2v + st);
      const bool on = b < a.B && mg > 0.f;  // hinge active (derivative 0 at margin 0)
      gsh[t] = on ? a.invB : 0.f;           // d loss/d s~ = m/B, d loss/d s = -m/B
      lossr = on ? mg : 0.f;
    }
  }
  if (SCORE) return;
  __syncthreads();

  // V and the db1 / dw2 sums of this lane's hidden units over its rows
  float db1[2] = {0.f, 0.f}, dw2[2] = {0.f, 0.f};
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int r = 16 * m + 4 * g + c, b = r0 + r;
      const float gst = gsh[r];
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const float hh = zh[m][n][c], hc = ht[m][n][c];
        // h - h~ = tanh(z - z~) (1 - h h~) with z - z~ = -D
        const float hmh = tanh_fast(-D[m][n][c]) * (1.f - hh * hc);
        const float gw = gst * w2v[n];
        const float dz = -gw * (1.f - hh * hh);
        const float dzt = gw * (1.f - hc * hc);
        const float dsum = gw * hmh * (hh + hc);
        if (b < a.B) {
          float* vr = a.V + (size_t)b * 3 * a.H + 32 * w + 16 * n + i;
          vr[0] = dsum;
          vr[a.H] = dz;
          vr[2 * a.H] = dzt;
          db1[n] += dsum;
          dw2[n] -= gst * hmh;  // -(m/B) h + (m/B) h~
        }
      }
    }
  float* vp = a.vpart + (size_t)blockIdx.x * (2 * a.H + 2);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    float x = db1[n], y = dw2[n];
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    if (g == 0) {
      vp[32 * w + 16 * n + i] = x;
      vp[a.H + 32 * w + 16 * n + i] = y;
    }
  }
  if (w == 0) {  // the workgroup's hinge sum (rows in order; R <= 64), db2 = 0
    for (int o = 1; o < kWave; o <<= 1) lossr += __shfl_xor(lossr, o);
    if (lane == 0) {
      vp[2 * a.H] = lossr;
      vp[2 * a.H + 1] = 0.f;
    }
  }
}

// =============================================================== dW1
//
// One workgroup per (64 CW columns of one window position or of the corrupt
// row, slice of the batch), all H = 64 HW hidden units; wave (wh, wc) owns a
// 64 x 64 block.  The contraction runs over the slice's windows, 32 a step:
// both operands need eight windows of one column per lane, so a thread reads
// a column of eight rows (adjacent threads, adjacent columns), splits it and
// stores whole fragments.  The next step's values are in flight in registers
// during a step.  The centre's true and corrupt halves are columns of their
// own (partial columns K .. K + d), so that every workgroup has the same
// work, and the slices are cut so that the workgroups fill the CUs once
// (large_dw1_slice).  Workgroups of one slice share its vectors: consecutive
// ones of the list go to one XCD (blocks go round the XCDs).
template <int HW, int CW>
__global__ __launch_bounds__(HW * CW * kWave) void k_large_dw1(LargeArgs a) {
  constexpr int H = 64 * HW, CB = 64 * CW, NT = HW * CW * kWave;
  constexpr int VU = 4 / CW;                      // V units (a column of 8 windows) per thread
  constexpr int XU = (4 + HW - 1) / HW;           // X units per thread
  constexpr int VF = (H / 16) * 3 * kWave, XF = (CB / 16) * 3 * kWave;
  extern __shared__ lu4 lds_q[];
  lu4* Vs = lds_q;                                // [2][VF]
  lu4* Xs = lds_q + 2 * VF;                       // [2][XF]
  int32_t* ids = reinterpret_cast<int32_t*>(Xs + 2 * XF);  // [slice]
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int wh = w % HW, wc = w / HW;
  if (2 * w >= HW * CW) __builtin_amdgcn_s_setprio(1);  // (as in k_large_fwd)
  const int d = a.d, ncol = (a.K + d) / CB, nwg = ncol * a.n_slices;
  const int per = (nwg + kXcds - 1) / kXcds;
  const int f = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
  if ((int)(blockIdx.x / kXcds) >= per || f >= nwg) return;
  const int sl = f / ncol, k0 = (f - sl * ncol) * CB;
  const int j = k0 / d, off0 = k0 - j * d;  // j == win: the corrupt row
  const int ty = j == a.win ? 2 : (j == a.c ? 1 : 0);
  const int b_lo = sl * a.slice, nb = min(a.B - b_lo, a.slice);
  const int steps = (nb + 31) / 32;

  for (int x = t; x < nb; x += NT) {
    const int32_t id = j == a.win ? a.corrupt[b_lo + x] : a.windows[(size_t)(b_lo + x) * a.win + j];
    ids[x] = (uint32_t)id < (uint32_t)a.V_rows ? id : 0;
  }
  __syncthreads();

  const float* vbase = a.V + (size_t)b_lo * 3 * H + (size_t)ty * H;
  // this thread's units: column vh of V, groups of eight windows vg, vg + CW, ..
  // and column xc of X, groups xg, xg + HW, .. (NT is CW H and HW CB; a wave's
  // groups are the same for its lanes)
  const int vh = t % H, vg = w / HW, xc = t % CB, xg = w / CW;
  float vr[VU][8], xr[XU][8];
  auto load_t = [&](auto tail, int st) LG_INLINE {  // tail: the step has windows past the slice
    constexpr bool TAIL = decltype(tail)::value;
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int r = 32 * st + 8 * (vg + CW * u);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int re = TAIL ? min(r + e, nb - 1) : r + e;
        vr[u][e] = vbase[re * 3 * H + vh];
        if (TAIL && r + e >= nb) vr[u][e] = 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int r = 32 * st + 8 * (xg + HW * u);
      if (4 % HW == 0 || xg + HW * u < 4) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int re = TAIL ? min(r + e, nb - 1) : r + e;
          xr[u][e] = a.E[(size_t)ids[re] * d + off0 + xc];
        }
      }
    }
  };
  auto load = [&](int st) LG_INLINE {
    if (32 * st + 32 <= nb) load_t(std::false_type{}, st);
    else load_t(std::true_type{}, st);
  };
  auto store = [&](int buf) LG_INLINE {
    float big = 0.f;
#pragma unroll
    for (int u = 0; u < VU; ++u) lg_largest(vr[u], big);
#pragma unroll
    for (int u = 0; u < XU; ++u)
      if (4 % HW == 0 || xg + HW * u < 4) lg_largest(xr[u], big);
    lg_checked(big, [&](auto safe) LG_INLINE {
      constexpr bool SAFE = decltype(safe)::value;
      lu4 p[3];
#pragma unroll
      for (int u = 0; u < VU; ++u) {
        lg_split8<SAFE>(vr[u], p);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          Vs[buf * VF + ((vh >> 4) * 3 + k) * kWave + 16 * (vg + CW * u) + (vh & 15)] = p[k];
      }
#pragma unroll
      for (int u = 0; u < XU; ++u) {
        if (4 % HW == 0 || xg + HW * u < 4) {
          lg_split8<SAFE>(xr[u], p);
#pragma unroll
          for (int k = 0; k < 3; ++k)
            Xs[buf * XF + ((xc >> 4) * 3 + k) * kWave + 16 * (xg + HW * u) + (xc & 15)] = p[k];
        }
      }
    });
  };
  f4 hi[4][4], lo[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) hi[m][n] = lo[m][n] = kZero4;
  load(0);
  store(0);
  if (steps > 1) load(1);
  __syncthreads();
  // step st reads buffer st & 1 and fills the other one, last read at step
  // st - 1, before its closing barrier.  The two waves of a SIMD stage at
  // opposite ends of the step, so that one splits while the other multiplies.
  auto stage = [&](int st) LG_INLINE {
    if (st + 1 < steps) store((st + 1) & 1);
    if (st + 2 < steps) load(st + 2);
  };
  for (int st = 0; st < steps; ++st) {
    const int buf = st & 1;
    if (2 * w < HW * CW) stage(st);
    const lu4* vs = Vs + buf * VF + wh * 4 * 3 * kWave + lane;
    const lu4* xs = Xs + buf * XF + wc * 4 * 3 * kWave + lane;
    lu4 A[4][3], Bv[2][3];
    lg_read<4>(vs, A);
    auto read_b = [&](int n, lu4 (&Bn)[3]) LG_INLINE {
#pragma unroll
      for (int k = 0; k < 3; ++k) Bn[k] = xs[(n * 3 + k) * kWave];
    };
    read_b(0, Bv[0]);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      if (n < 3) read_b(n + 1, Bv[(n + 1) & 1]);
      lg_pin();
      const lu4 (&Bn)[3] = Bv[n & 1];
      constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
      for (int p = 0; p < 5; ++p)
#pragma unroll
        for (int m = 0; m < 4; ++m) lo[m][n] = lg_mfma(A[m][PA[p]], Bn[PB[p]], lo[m][n]);
#pragma unroll
      for (int m = 0; m < 4; ++m) hi[m][n] = lg_mfma(A[m][0], Bn[0], hi[m][n]);
      lg_pin();
    }
    if (2 * w >= HW * CW) stage(st);
    __syncthreads();
  }
  // lane (i, g), component r: hidden 64 wh + 16m + 4g + r, column k0 + 64 wc + 16n + i
  const int Kx = a.K + d, i = lane & 15, g = lane >> 4;
  float* P = a.part + (size_t)sl * H * Kx;
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const f4 v = lg_sum(hi[m][n], lo[m][n]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        P[(size_t)(64 * wh + 16 * m + 4 * g + r) * Kx + k0 + 64 * wc + 16 * n + i] = v[r];
    }
}

// =============================================================== G
//
// A workgroup takes 64 windows and a range of the entry positions (all of
// them when the windows alone fill the CUs), ordered context positions, true
// centre, corrupt.  The windows' vectors of one type sit in LDS as A fragments
// for every position that uses them.  Wave (cg, pg) owns 32 columns and takes every PG-th
// context position whole (64 x 32 outputs); positions left over, and the two
// centre entries, are split by windows over the PG groups.  W1's fragments
// belong to one wave each and come straight from memory, a step ahead.
template <int CG, int PG>
__global__ __launch_bounds__(CG * PG * kWave) void k_large_g(LargeArgs a) {
  constexpr int NT = CG * PG * kWave, D = 32 * CG;
  constexpr int UPT = (kLgGRows * (kMaxLargeH / 8) + NT - 1) / NT;  // staged units per thread
  extern __shared__ lu4 lds_q[];  // [H/32 steps][4 row tiles][3][64]
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int cg = w % CG, pg = w / CG, i = lane & 15, g = lane >> 4;
  if (2 * w >= CG * PG) __builtin_amdgcn_s_setprio(1);  // (as in k_large_fwd)
  const int b0 = blockIdx.x * kLgGRows, ns = a.H / 32, W1p = a.win + 1;
  const int o_lo = (int)((int64_t)blockIdx.y * W1p / gridDim.y);
  const int o_hi = (int)((int64_t)(blockIdx.y + 1) * W1p / gridDim.y);
  const int nctx = a.win - 1;  // context positions come first

  // unit u: windows 16 (u / 64 % 4) + (u & 15), hidden units 8g.. of step u / 256
  f4 vr[UPT][2];
  auto load = [&](int ty) LG_INLINE {
#pragma unroll
    for (int v = 0; v < UPT; ++v) {
      const int u = t + v * NT, s = u >> 6;
      const int b = b0 + 16 * (s & 3) + (u & 15);
      vr[v][0] = vr[v][1] = kZero4;
      if (s < 4 * ns && b < a.B) {
        const float* src = a.V + ((size_t)b * 3 + ty) * a.H + 32 * (s >> 2) + 8 * ((u >> 4) & 3);
        vr[v][0] = ld4(src);
        vr[v][1] = ld4(src + 4);
      }
    }
  };
  auto store = [&]() LG_INLINE {
    float big = 0.f;
#pragma unroll
    for (int v = 0; v < UPT; ++v)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float x[4] = {vr[v][k][0], vr[v][k][1], vr[v][k][2], vr[v][k][3]};
        lg_largest(x, big);
      }
    lg_checked(big, [&](auto safe) LG_INLINE {
#pragma unroll
      for (int v = 0; v < UPT; ++v) {
        const int u = t + v * NT, s = u >> 6;
        if (s < 4 * ns) {
          float x[8];
          lu4 p[3];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = vr[v][e >> 2][e & 3];
          lg_split8<decltype(safe)::value>(x, p);
#pragma unroll
          for (int k = 0; k < 3; ++k) lds_q[(s * 3 + k) * kWave + (u & 63)] = p[k];
        }
      }
    });
  };
  auto load_w = [&](int jj, int hs, lu4 (&Bv)[2][3]) LG_INLINE {
    const lu4* src = a.wg + ((size_t)(jj * (D / 16) + 2 * cg) * ns + hs) * 3 * kWave + lane;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int k = 0; k < 3; ++k) Bv[n][k] = src[((size_t)n * ns * 3 + k) * kWave];
  };
  // position o of the order: entry position and W1 block
  auto entry = [&](int o) LG_INLINE { return o < nctx ? o + (o >= a.c) : (o == nctx ? a.c : a.win); };
  auto block = [&](int o) LG_INLINE { return o < nctx ? o + (o >= a.c) : a.c; };
  lu4 B0[2][3], B1[2][3];
  // output rows [16 m0, 16 (m0 + MT)) of position o, whose first two steps'
  // fragments are loaded; loads those of position on (if >= 0) at the end
  auto compute = [&](auto mt_c, int m0, int o, int on) LG_INLINE {
    constexpr int MT = decltype(mt_c)::value;
    f4 hi[MT][2], lo[MT][2];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) hi[m][n] = lo[m][n] = kZero4;
    const int jj = block(o), jn = on >= 0 ? block(on) : -1;
    auto step = [&](int hs, lu4 (&Bv)[2][3]) LG_INLINE {
      lg_step<MT>(lds_q + (hs * 4 + m0) * 3 * kWave + lane, Bv, hi, lo);
      if (hs + 2 < ns) load_w(jj, hs + 2, Bv);
      else if (jn >= 0) load_w(jn, hs + 2 - ns, Bv);
    };
    for (int hs = 0; hs < ns; hs += 2) {  // ns is even
      step(hs, B0);
      step(hs + 1, B1);
    }
    const int j = entry(o);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const f4 v = lg_sum(hi[m][n], lo[m][n]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int b = b0 + 16 * (m0 + m) + 4 * g + c;
          if (b < a.B) a.G[((size_t)b * W1p + j) * D + 32 * cg + 16 * n + i] = v[c];
        }
      }
  };
  constexpr int MS = 4 / PG;  // row tiles of a wave in a position split by windows
  const int c_hi = min(o_hi, nctx);
  const int whole = o_lo < c_hi ? (c_hi - o_lo) / PG * PG : 0;  // positions taken whole
  const int o_s = o_lo + whole;                                 // first one split by windows
  // this wave's positions in order: o_lo + pg, + PG, ... below o_s, then o_s .. o_hi - 1
  auto next_of = [&](int o) LG_INLINE {
    const int nx = o < o_s ? (o + PG < o_s ? o + PG : o_s) : o + 1;
    return nx < o_hi ? nx : -1;
  };
  auto type_of = [&](int o) LG_INLINE { return o < nctx ? 0 : (o == nctx ? 1 : 2); };
  int o = whole > 0 ? o_lo + pg : o_s;
  load_w(block(o), 0, B0);
  load_w(block(o), 1, B1);
  load(type_of(o_lo));
  store();
  __syncthreads();
  int ty = type_of(o_lo);
  while (o >= 0) {
    if (type_of(o) != ty) {  // every wave reaches a new type at the same position
      __syncthreads();
      load(ty + 1);
      store();
      __syncthreads();
      ++ty;
    }
    const int on = next_of(o);
    if (PG == 1 || o < o_s) compute(std::integral_constant<int, 4>{}, 0, o, on);
    else compute(std::integral_constant<int, MS>{}, MS * pg, o, on);
    o = on;
  }
}

}  // namespace pg
