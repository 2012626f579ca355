// Score, gather and index-check kernels.
#pragma once
#include "common.h"
#include "fwdbwd_dev.h"
#include "launch.h"

namespace pg {

// =============================================================== score

template <int NT, int CPW>
__global__ __launch_bounds__(kBlock) void k_score(ScoreArgs a) {
  extern __shared__ uint32_t lds[];
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int n16 = lane & 15, g = lane >> 4;
  const int dq = a.d / 16, nchunk = a.K / 16;
  int32_t* ids = reinterpret_cast<int32_t*>(lds);                  // [16][win]
  int32_t* badrow = ids + kTileRows * kMaxWin;                      // [16]
  f4* zp = reinterpret_cast<f4*>(lds + kTileRows * (kMaxWin + 1));  // [4][NT][64]
  const int row0 = blockIdx.x * kTileRows;
  if (t < kTileRows) badrow[t] = 0;
  __syncthreads();
  for (int i = t; i < kTileRows * a.win; i += kBlock) {
    const int r = i / a.win, j = i - r * a.win;
    const int b = row0 + r;
    const int32_t id = b < a.B ? a.windows[(size_t)b * a.win + j] : 0;
    const bool bad = (uint32_t)id >= (uint32_t)a.V;
    if (bad) {
      atomicOr(a.flag, kFlagBadId);
      badrow[r] = 1;
    }
    ids[i] = bad ? 0 : id;
  }
  __syncthreads();
  f4 x[CPW], wv[CPW][NT];
#pragma unroll
  for (int ci = 0; ci < CPW; ++ci) {
    const int kc = w + kWavesPerBlock * ci;
    const bool ok = kc < nchunk;
    const int j = ok ? kc / dq : 0;
    const int off = (kc - j * dq) * 16 + 4 * g;
    x[ci] = ok ? ld4(a.E + (size_t)ids[n16 * a.win + j] * a.d + off) : kZero4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int n = nt * 16 + n16;
      wv[ci][nt] = (ok && n < a.H) ? ld4(a.W1 + (size_t)n * a.K + kc * 16 + 4 * g) : kZero4;
    }
  }
  f4 z[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) z[nt] = kZero4;
#pragma unroll
  for (int ci = 0; ci < CPW; ++ci)
    if (w + kWavesPerBlock * ci < nchunk)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) z[nt] = mfma16(x[ci][q], wv[ci][nt][q], z[nt]);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) zp[(w * NT + nt) * kWave + lane] = z[nt];
  __syncthreads();
  if (w != 0) return;
  float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    f4 Z = zp[(0 * NT + nt) * kWave + lane];
#pragma unroll
    for (int v = 1; v < kWavesPerBlock; ++v) Z += zp[(v * NT + nt) * kWave + lane];
    const int n = nt * 16 + n16;
    const float b1v = n < a.H ? a.b1[n] : 0.f, w2v = n < a.H ? a.w2[n] : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) ps[i] += w2v * tanh_fast(b1v + Z[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) ps[i] += __shfl_xor(ps[i], o);
  if (n16 == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * g + i, b = row0 + r;
      if (b < a.B) a.scores[b] = badrow[r] ? __builtin_nanf("") : a.b2[0] + ps[i];
    }
  }
}

// =============================================================== gather
//
// A wave copies a.rows consecutive entries (rows of X and Xc): each lane looks
// up one entry, and the rows then go as one flat list of 16-byte words,
// U of them in flight per lane.  An entry's position is divided out once per row
// and not once per word, and by 32-bit arithmetic.
//
// NT: non-temporal stores, for outputs that the L2s cannot hold (kGatherKeep):
// X is written once and several times the size of the rows read, which would
// lose their place in the caches to it.  Smaller outputs are left there for
// whoever reads X next, and two words per lane in flight fill the chip as well
// as eight.  us per call alone | followed by an addition over X | by a product of
// X with 64 columns, calls in a graph, non-temporal and eight words against plain
// and two (outputs; rows of 64 or 128):
//     0.8 MB   3.0, 2.6 |  5.1,  4.4 | 11.4,  9.0
//     6.3 MB   3.7, 3.5 |  8.1,  7.6 | 13.7, 11.4
//    12.6 MB   4.3, 4.7 | 11.8, 11.7 | 16.4, 14.3
//    25.2 MB   6.6, 7.2 | 18.1, 16.6 | 23.6, 19.1 (rows of 64)
//    25.2 MB   6.6, 7.3 | 19.6, 16.7 | 27.5, 21.9 (rows of 128)
//    50.3 MB  11.2, 13.2 | 28.8, 26.8 | 30.6, 29.7
//   100.7 MB  24.4, 25.4 | 53.9, 55.8 | 53.1, 52.4
// 65,536 windows of 5 rows of 64 (100.7 MB), three outputs in turn: a thread per
// word with two 64-bit divisions 34.6 us, eight words with plain stores 31.7,
// non-temporal 22.0.
constexpr size_t kGatherKeep = (size_t)32 << 20;  // bytes: the eight L2s of 4 MB

template <int U, bool NT>
__global__ __launch_bounds__(kBlock) void k_gather(GatherArgs a) {
  __shared__ int2 ent[kWavesPerBlock][kWave];  // (id or -1, row of X or ~row of Xc)
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int q4 = a.d / 4, W1p = a.win + 1;
  const int N = a.B * W1p;
  const int e0 = (blockIdx.x * kWavesPerBlock + w) * a.rows;
  const int nr = min(a.rows, N - e0);
  if (nr <= 0) return;
  if (lane < nr) {
    const int e = e0 + lane, b = e / W1p, j = e - b * W1p;
    int32_t id = j < a.win ? a.windows[e - b] : a.corrupt[b];  // b win + j = e - b
    if ((uint32_t)id >= (uint32_t)a.V) {
      atomicOr(a.flag, kFlagBadId);
      id = -1;
    }
    ent[w][lane] = int2{id, j < a.win ? e - b : ~b};
  }
  wave_lds_sync();
  const int total = nr * q4;
  for (int f0 = lane; f0 < total; f0 += kWave * U) {
    f4 v[U];
    float* dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = min(f0 + u * kWave, total - 1);
      const int r = (int)((uint32_t)f * a.rq4 >> 20), q = f - r * q4;  // f / q4: f < 4096
      const int2 x = ent[w][r];
      dst[u] = x.y >= 0 ? a.X + (size_t)x.y * a.d + 4 * q : a.Xc + (size_t)~x.y * a.d + 4 * q;
      const float nan = __builtin_nanf("");
      v[u] = f4{nan, nan, nan, nan};
      if (x.x >= 0) v[u] = ld4(a.E + (size_t)x.x * a.d + 4 * q);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (f0 + u * kWave < total) {
        if constexpr (NT) __builtin_nontemporal_store(v[u], reinterpret_cast<f4*>(dst[u]));
        else st4(dst[u], v[u]);
      }
  }
}

// =============================================================== index check

__global__ __launch_bounds__(kBlock) void k_check_idx(const int32_t* idx, int N, int rows,
                                                      uint32_t* flag) {
  bool bad = false;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < N; i += gridDim.x * kBlock)
    bad |= (uint32_t)idx[i] >= (uint32_t)rows;
  if (bad) atomicOr(flag, kFlagBadId);
}


}  // namespace pg
