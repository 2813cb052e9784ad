// Block-granular variant of the KV selection (paper Sec. "Block-wise probing and sparse flash attention
// kernel", the way the paper runs it): queries AND keys are mean-pooled along the sequence in blocks, the
// pooled attention map gives one accumulated score per key block, the recall budget is a number of
// blocks, and the selected blocks are handed to the attention kernels as token lists.
//
//  * pool_rows_kernel: block means of the rows of one head, fp32 (HBM-bound, one pass over Q and K).
//  * block_rows_kernel, block_cols_kernel: the pooled map twice, by rows for every row's softmax statistics, then by
//    columns for a[m] = sum_j w_j P_j[m] (a key block of c tokens weighs c in a row), in a fixed order without atomics.
//  * expand_blocks_kernel: ascending block ids -> ascending token ids (tokens past the end of the sequence
//    in a partial last block become pad entries, which the packers turn into zero rows nobody sees).
#include "common.h"
#include "kernels.h"

namespace omni {

namespace {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

// grid: (n_blocks, B * H).  X is [B, H, N, D] with element strides sb, sh, sn.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void pool_rows_kernel(const T* __restrict__ X, long long sb, long long sh,
                                                            long long sn, int H, int N, int block, int nblk,
                                                            float* __restrict__ out) {
  constexpr int E = Elem<T>::kPer16B;
  constexpr int LPR = D / E;
  constexpr int RPP = kThreads / LPR;
  __shared__ float red[RPP][D];
  const int j = blockIdx.x, bh = blockIdx.y;
  const int b = bh / H, i = bh % H;
  const T* base = X + b * sb + i * sh;
  const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR;
  const int row_begin = j * block, row_end = min(N, row_begin + block);
  float acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;
  for (int r = row_begin + r0; r < row_end; r += RPP) {
    const u32x4 raw = *reinterpret_cast<const u32x4*>(base + (long long)r * sn + c * E);
    float v[E];
    unpack16(raw, v, (const T*)nullptr);
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] += v[e];
  }
#pragma unroll
  for (int e = 0; e < E; ++e) red[r0][c * E + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
    for (int r = 0; r < RPP; ++r) s += red[r][threadIdx.x];
    out[((long long)bh * nblk + j) * D + threadIdx.x] = s / (float)(row_end - row_begin);
  }
}

// The pooled map has n_blocks^2 logits of D products per head: little work, so what counts is how many workgroups share
// it and how long a thread's chain of dependent multiply-adds is.  Every thread keeps one key block and forms the logits
// of several query blocks side by side; the map is formed twice, which is cheaper than keeping it (4 n_blocks^2 bytes a
// head).  One workgroup per head walking its rows one after the other took 251 us at 64 blocks, 28 heads, d = 128; the two
// kernels take 18 + 22.
constexpr int kRowsPerWg = 8;                // query blocks of a row workgroup
constexpr int kColsPerWg = 32;               // key blocks of a column workgroup ...
constexpr int kColSlices = kThreads / kColsPerWg;   // ... whose rows are dealt to this many slices
constexpr int kColBatch = 4;                 // rows a thread forms side by side
constexpr int kMaxBlocks = 2048;

// dot[r] = q row r . k, in the order of d, for R rows of sq (LDS, D floats each)
template <int D, int R>
__device__ __forceinline__ void dots(const float* sq, const float* __restrict__ k, float (&dot)[R]) {
#pragma unroll
  for (int r = 0; r < R; ++r) dot[r] = 0.f;
#pragma unroll 4
  for (int d = 0; d < D; d += 4) {
    const f32x4 kv = *reinterpret_cast<const f32x4*>(k + d);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const f32x4 qv = *reinterpret_cast<const f32x4*>(sq + r * D + d);
#pragma unroll
      for (int e = 0; e < 4; ++e) dot[r] = fmaf(qv[e], kv[e], dot[r]);
    }
  }
}

// tokens of block m
__device__ __forceinline__ float block_tokens(int m, int block, int N) { return (float)(min(N, (m + 1) * block) - m * block); }

// grid: (cdiv(n_blocks, kRowsPerWg), B * Hq).  Of every pooled row: the largest logit and (queries of the block) /
// (sum of the key blocks' weights against it).
template <int D>
__global__ __launch_bounds__(kThreads) void block_rows_kernel(const float* __restrict__ qbar, const float* __restrict__ kbar,
                                                             int Hq, int Hkv, int N, int block, int nblk, int causal,
                                                             float scale, float2* __restrict__ stats) {
  __shared__ __attribute__((aligned(16))) float sq[kRowsPerWg * D];
  __shared__ float sm[kRowsPerWg][kThreads / 64], ss[kRowsPerWg][kThreads / 64];
  const int bh = blockIdx.y, b = bh / Hq, i = bh % Hq, g = i / (Hq / Hkv), j0 = blockIdx.x * kRowsPerWg;
  const float* qh = qbar + ((long long)bh * nblk + j0) * D;
  const float* kh = kbar + (long long)(b * Hkv + g) * nblk * D;
  const float c2 = scale * kLog2e;
  const int rows = min(kRowsPerWg, nblk - j0);
  for (int t = threadIdx.x; t < kRowsPerWg * D; t += kThreads) sq[t] = t < rows * D ? qh[t] : 0.f;
  __syncthreads();
  float mx[kRowsPerWg], sum[kRowsPerWg];
#pragma unroll
  for (int r = 0; r < kRowsPerWg; ++r) mx[r] = -INFINITY, sum[r] = 0.f;
  const int end = causal ? j0 + rows : nblk;       // no row of this workgroup sees a key block past this
  for (int m = threadIdx.x; m < end; m += kThreads) {
    float dot[kRowsPerWg];
    dots<D, kRowsPerWg>(sq, kh + (long long)m * D, dot);
    const float cm = block_tokens(m, block, N);
#pragma unroll
    for (int r = 0; r < kRowsPerWg; ++r) {
      const float l = dot[r] * c2, top = fmaxf(mx[r], l);
      if ((causal && m > j0 + r) || l == -INFINITY) continue;      // no weight (and no maximum to compare with)
      sum[r] = sum[r] * exp2f(mx[r] - top) + cm * exp2f(l - top);
      mx[r] = top;
    }
  }
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < kRowsPerWg; ++r) {
    const float top = wave_max(mx[r]);
    const float part = wave_sum(sum[r] == 0.f ? 0.f : sum[r] * exp2f(mx[r] - top));    // a NaN logit stays in the sum
    if (lane_id() == 0) sm[r][wave] = top, ss[r][wave] = part;
  }
  __syncthreads();
  if ((int)threadIdx.x < rows) {
    const int r = threadIdx.x;
    float top = sm[r][0], part = 0.f;
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) top = fmaxf(top, sm[r][w]);
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) part += ss[r][w] == 0.f ? 0.f : ss[r][w] * exp2f(sm[r][w] - top);
    stats[(long long)bh * nblk + j0 + r] = make_float2(top, block_tokens(j0 + r, block, N) / part);
  }
}

// grid: (cdiv(n_blocks, kColsPerWg), B * Hq).  Column sums; slice s of a column takes the rows of its own batches, the
// slices are added in order.
template <int D>
__global__ __launch_bounds__(kThreads) void block_cols_kernel(const float* __restrict__ qbar, const float* __restrict__ kbar,
                                                             int Hq, int Hkv, int N, int block, int nblk, int causal,
                                                             float scale, const float2* __restrict__ stats,
                                                             float* __restrict__ out) {
  constexpr int kTrip = kColSlices * kColBatch;    // rows staged per trip
  __shared__ __attribute__((aligned(16))) float sq[kTrip * D];
  __shared__ float2 sst[kTrip];
  __shared__ float sacc[kColSlices][kColsPerWg];
  const int bh = blockIdx.y, b = bh / Hq, i = bh % Hq, g = i / (Hq / Hkv);
  const int col = threadIdx.x % kColsPerWg, slice = threadIdx.x / kColsPerWg, m = blockIdx.x * kColsPerWg + col;
  const float* qh = qbar + (long long)bh * nblk * D;
  const float* kr = kbar + ((long long)(b * Hkv + g) * nblk + min(m, nblk - 1)) * D;
  const float c2 = scale * kLog2e, cm = m < nblk ? block_tokens(m, block, N) : 0.f;
  float acc = 0.f;
  const int begin = causal ? (int)blockIdx.x * kColsPerWg / kTrip * kTrip : 0;    // earlier rows see none of these columns
  for (int j0 = begin; j0 < nblk; j0 += kTrip) {
    __syncthreads();
    const int rows = min(kTrip, nblk - j0);
    for (int t = threadIdx.x; t < kTrip * D; t += kThreads) sq[t] = t < rows * D ? qh[(long long)j0 * D + t] : 0.f;
    if (threadIdx.x < kTrip)
      sst[threadIdx.x] = (int)threadIdx.x < rows ? stats[(long long)bh * nblk + j0 + threadIdx.x] : make_float2(0.f, 0.f);
    __syncthreads();
    float dot[kColBatch];
    dots<D, kColBatch>(sq + slice * kColBatch * D, kr, dot);
#pragma unroll
    for (int r = 0; r < kColBatch; ++r) {
      const int j = j0 + slice * kColBatch + r;
      const float2 st = sst[slice * kColBatch + r];
      if (j < nblk && (!causal || m <= j)) acc = fmaf(st.y, cm * exp2f(dot[r] * c2 - st.x), acc);
    }
  }
  sacc[slice][col] = acc;
  __syncthreads();
  if (threadIdx.x < kColsPerWg && m < nblk) {
    float a = 0.f;
#pragma unroll
    for (int s = 0; s < kColSlices; ++s) a += sacc[s][col];
    out[(long long)bh * nblk + m] = a * ((float)nblk / (float)N);        // scores sum to the number of blocks
  }
}

// grid: (cdiv(blk_cap * block, 256), B * Hq).  tile_map (block % 64 == 0), if wanted: [B*Hq, blk_cap * block / 64] tile of the
// KV head's token-ordered K/V that holds tile t of the head's key list.
__global__ __launch_bounds__(256) void expand_blocks_kernel(const int* __restrict__ blk_idx, const int* __restrict__ blk_budget,
                                                            int Hq, int blk_cap, int block, int N, int b_cap,
                                                            int* __restrict__ kv_idx, int* __restrict__ budget,
                                                            int last_tile, int* __restrict__ tile_map) {
  const int bh = blockIdx.y, b = bh / Hq;
  const int nb = min(blk_budget[b], blk_cap);
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (bh % Hq == 0 && t == 0) budget[b] = min(nb * block, b_cap);
  if (tile_map && t % kTileN == 0 && t < blk_cap * block) {
    const int at = t < nb * block ? min((blk_idx[(long long)bh * blk_cap + t / block] * block + t % block) / kTileN, last_tile) : 0;
    tile_map[((long long)bh * blk_cap * block + t) / kTileN] = at;
  }
  if (t >= nb * block || t >= b_cap) return;
  const int tok = blk_idx[(long long)bh * blk_cap + t / block] * block + t % block;
  kv_idx[(long long)bh * b_cap + t] = tok < N ? tok : kPadKeyIndex;
}

struct BlockWs {
  float* qbar;
  float* kbar;
  float2* stats;
};

BlockWs carve_block(Arena& a, const Layer& L, int nblk) {
  BlockWs w;
  w.qbar = a.take<float>((size_t)L.B * L.Hq * nblk * L.D);
  w.kbar = a.take<float>((size_t)L.B * L.Hkv * nblk * L.D);
  w.stats = a.take<float2>((size_t)L.B * L.Hq * nblk);
  return w;
}

template <typename T, int D>
int launch_block_scores(const Layer& L, const void* Q, const void* K, int block, float* out, void* ws, hipStream_t st) {
  const int nblk = cdiv(L.N, block);
  Arena a(ws);
  BlockWs w = carve_block(a, L, nblk);
  hipLaunchKernelGGL((pool_rows_kernel<T, D>), dim3(nblk, L.B * L.Hq), dim3(kThreads), 0, st, static_cast<const T*>(Q),
                     L.qs[0], L.qs[1], L.qs[2], L.Hq, L.N, block, nblk, w.qbar);
  OMNI_LAUNCH_CHECK();
  hipLaunchKernelGGL((pool_rows_kernel<T, D>), dim3(nblk, L.B * L.Hkv), dim3(kThreads), 0, st, static_cast<const T*>(K),
                     L.ks[0], L.ks[1], L.ks[2], L.Hkv, L.N, block, nblk, w.kbar);
  OMNI_LAUNCH_CHECK();
  hipLaunchKernelGGL((block_rows_kernel<D>), dim3(cdiv(nblk, kRowsPerWg), L.B * L.Hq), dim3(kThreads), 0, st, w.qbar, w.kbar,
                     L.Hq, L.Hkv, L.N, block, nblk, L.causal, L.scale, w.stats);
  OMNI_LAUNCH_CHECK();
  hipLaunchKernelGGL((block_cols_kernel<D>), dim3(cdiv(nblk, kColsPerWg), L.B * L.Hq), dim3(kThreads), 0, st, w.qbar, w.kbar,
                     L.Hq, L.Hkv, L.N, block, nblk, L.causal, L.scale, w.stats, out);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

}  // namespace

int block_scores_max_blocks() { return kMaxBlocks; }

size_t block_scores_ws(const Layer& L, int block) {
  Arena a(nullptr);
  carve_block(a, L, cdiv(L.N, block));
  return a.used();
}

int run_block_scores(const Layer& L, int dtype, const void* Q, const void* K, int block, float* out, void* ws,
                     hipStream_t st) {
  if (dtype == OMNI_BF16) {
    if (L.D == 128) return launch_block_scores<u16, 128>(L, Q, K, block, out, ws, st);
    return launch_block_scores<u16, 64>(L, Q, K, block, out, ws, st);
  }
  if (L.D == 128) return launch_block_scores<float, 128>(L, Q, K, block, out, ws, st);
  return launch_block_scores<float, 64>(L, Q, K, block, out, ws, st);
}

int run_expand_blocks(const Layer& L, const int* blk_idx, const int* blk_budget, int blk_cap, int block, int* kv_idx,
                      int* budget, int b_cap, hipStream_t st, int* tile_map, int last_tile) {
  hipLaunchKernelGGL(expand_blocks_kernel, dim3(cdiv((long long)blk_cap * block, 256LL), L.B * L.Hq), dim3(256), 0, st,
                     blk_idx, blk_budget, L.Hq, blk_cap, block, L.N, b_cap, kv_idx, budget, last_tile, tile_map);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

}  // namespace omni
