// Device code of the probe keys and of the lazy/active scores (score.hip) that other launches of a short selection take in.
#pragma once

#include "common.h"

namespace omni {

constexpr int kScoreThreads = 256;
constexpr int kMeanRowsPerChunk = 256;     // ~1000 workgroups at 64k: enough to fill the memory system
constexpr int kFinalSplit = 8;             // interleaved partial sums per element of the mean, added in a fixed order

namespace {

// Sum of the visual keys of chunk `chunk` of KV head bg.  red: kScoreThreads / lanes per row x D floats.
template <typename T, int D>
__device__ __forceinline__ void mean_key_block(const T* __restrict__ K, const Layer& L, const Ragged& rg, int nchunk, int chunk,
                                               int bg, float* __restrict__ partial, float* red_) {
  constexpr int E = Elem<T>::kPer16B;
  constexpr int LPR = D / E;              // lanes per row
  constexpr int RPP = kScoreThreads / LPR;     // rows per pass
  float (*red)[D] = reinterpret_cast<float (*)[D]>(red_);
  const int b = bg / L.Hkv, g = bg % L.Hkv;
  const T* base = K + b * L.ks[0] + g * L.ks[1];
  const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR;
  const int v1 = rg.on ? rg.v1[b] : L.v1;
  const int row_begin = (rg.on ? rg.v0[b] : L.v0) + chunk * kMeanRowsPerChunk;
  const int row_end = min(v1, row_begin + kMeanRowsPerChunk);
  if (row_begin >= v1) return;             // a shorter sequence of a padded batch
  float acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;
  constexpr int kRowsInFlight = 8;         // loads issued together; added in ascending order of the rows
  for (int rb = row_begin + r0; rb < row_end; rb += RPP * kRowsInFlight) {
    u32x4 raw[kRowsInFlight];
#pragma unroll
    for (int u = 0; u < kRowsInFlight; ++u) {
      const int r = rb + u * RPP;
      if (r < row_end) raw[u] = *reinterpret_cast<const u32x4*>(base + (long long)r * L.ks[2] + c * E);
    }
#pragma unroll
    for (int u = 0; u < kRowsInFlight; ++u) {
      if (rb + u * RPP >= row_end) break;
      float v[E];
      unpack16(raw[u], v, (const T*)nullptr);
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] += v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) red[r0][c * E + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
#pragma unroll 4
    for (int r = 0; r < RPP; ++r) s += red[r][threadIdx.x];
    partial[((long long)bg * nchunk + chunk) * D + threadIdx.x] = s;
  }
}

// score = softmax([q.k_lazy, q.k_act] * scale)[1] = 1 / (1 + exp(-(q.(k_act - k_lazy)) * scale)) of kScoreRows rows of head bh, with
// the mean of the visual keys from its chunks' sums; the first block of a KV group's first head writes the probe keys.  The rows'
// scores end up one in every lane of the row's lane group, so that the exponential is evaluated (and its code fetched) once.
// diffs: D floats of LDS.
constexpr int kScoreRows = 128;
template <typename T, int D>
__device__ __forceinline__ void score_rows_block(const T* __restrict__ Q, const T* __restrict__ K, const Layer& L, const Ragged& rg,
                                                 int nchunk, const float* __restrict__ partial, int block, int bh,
                                                 float* __restrict__ probe, float* __restrict__ scores, float* diffs) {
  constexpr int E = Elem<T>::kPer16B;
  constexpr int LPR = D / E, RPP = kScoreThreads / LPR, kInFlight = kScoreRows / RPP;
  static_assert(kInFlight <= LPR, "a score per lane");
  const int b = bh / L.Hq, i = bh % L.Hq, g = i / L.G, bg = b * L.Hkv + g;
  const int N = seq_len(L, rg, b), row0 = block * kScoreRows;
  if (row0 >= N) return;
  const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR;
  const T* base = Q + b * L.qs[0] + i * L.qs[1] + c * E;
  u32x4 raw[kInFlight];
#pragma unroll
  for (int u = 0; u < kInFlight; ++u)
    raw[u] = *reinterpret_cast<const u32x4*>(base + (long long)min(row0 + u * RPP + r0, N - 1) * L.qs[2]);
  if (threadIdx.x < D) {
    const int n_vis = rg.on ? rg.v1[b] - rg.v0[b] : L.v1 - L.v0, chunks = cdiv(n_vis, kMeanRowsPerChunk);
    float part[kFinalSplit];
#pragma unroll
    for (int k = 0; k < kFinalSplit; ++k) part[k] = 0.f;
#pragma unroll 1
    for (int c0 = 0; c0 < chunks; c0 += kFinalSplit) {
#pragma unroll
      for (int k = 0; k < kFinalSplit; ++k) {
        const float x = partial[((long long)bg * nchunk + min(c0 + k, chunks - 1)) * D + threadIdx.x];
        part[k] += c0 + k < chunks ? x : 0.f;
      }
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < kFinalSplit; ++k) s += part[k];
    const float lazy = Elem<T>::load(K + b * L.ks[0] + g * L.ks[1] + (long long)L.sink * L.ks[2] + threadIdx.x);
    const float act = s / (float)n_vis;
    if (block == 0 && i % L.G == 0) {
      probe[((long long)bg * 2 + 0) * D + threadIdx.x] = lazy;
      probe[((long long)bg * 2 + 1) * D + threadIdx.x] = act;
    }
    diffs[threadIdx.x] = act - lazy;
  }
  __syncthreads();
  float mine = 0.f;
#pragma unroll
  for (int u = 0; u < kInFlight; ++u) {
    float v[E], dot = 0.f;
    unpack16(raw[u], v, (const T*)nullptr);
#pragma unroll
    for (int e = 0; e < E; ++e) dot = fmaf(v[e], diffs[c * E + e], dot);
    dot = row_lanes_sum<LPR>(dot);
    mine = c == u ? dot : mine;
  }
  const int row = row0 + c * RPP + r0;
  if (c < kInFlight && row < N) scores[(long long)bh * L.ld + row] = 1.0f / (1.0f + expf(-mine * L.scale));
}

}  // namespace

}  // namespace omni
