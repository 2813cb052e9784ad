// Backward of the sparse attention (omni_sparse_attn_bwd): gradients of
// O = softmax(Q K^T scale) V over kept queries x selected keys with the index
// sets held constant (the paper trains with the same sparse attention and gives
// no gradient through the selection):
//   P = exp(S - lse), dV = P^T dO, dP = dO V^T, dS = P (dP - delta),
//   delta = rowsum(dO O), dQ = scale dS K, dK = scale dS^T Q.
//
// Deterministic, no floating-point atomics.  bf16 (the measured path), two kernels in the forward's style
// (8 wavefronts, LDS-DMA ring, position masks from the visible-prefix counts):
//  * attn_bwd_bf16_kernel, persistent, goes through two lists one after the other.
//    Key items: 256 packed keys of a query head (32 per wavefront, K and V fragments resident); 32-query tiles (d = 64: 64) of
//    the packed kept rows (Q, dO in fragment order and k-packed, lse and delta by 4-byte LDS-DMA) are streamed: S = Q K^T,
//    dP = dO V^T, dV' += P^T dO, dK' += dS^T Q.  A key tile seen by many query tiles is shared by up to four workgroups,
//    each with a partial plane of its own.
//    dQ items: 256 kept queries of a head (32 per wavefront) from the forward's longest-first list; 64-key tiles of K, V
//    (fragment order) and K^T (k-packed): S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T.  Where the rows are few, 32 kept queries
//    whose keys the eight wavefronts share.
//  * attn_bwd_reduce_kernel adds the per-query-head dK', dV' rows (and split planes) of a KV group in a fixed order
//    into dK, dV -- a head's row is found through an inverse slot map -- and writes zeros for unselected tokens.
// fp32 inputs, on the fp32 32x32x2 MFMA: attn_bwd_f32_kernel (blocks for dK' and dV' of 32 keys, and for dQ);
// on long sequences attn_bwd_key_f32_long_kernel (128 keys) and attn_bwd_dq_f32_long_kernel (128 queries of the work list).
#include <algorithm>

#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "sched.h"

namespace omni {

namespace {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

struct BwdParams {
  const void* Q;
  const void* dO;
  Layer L;
  const int* q_idx;
  const int* q_cnt;
  const int* budget;
  int b_cap, npad, nqpad;
  const void* Kn;       // packed K, V in fragment order (fp32 on long sequences: row by row)
  const void* Vn;
  const void* Kt;       // k-packed K
  const void* Qt;       // k-packed kept Q, dO (these and the next two, and Kt: not for fp32 on long sequences)
  const void* dOt;
  const void* Qn;       // kept Q, dO rows in kept order, in fragment order
  const void* dOn;
  const float* lse2c;   // per kept position: lse * log2e (+inf: contributes nothing)
  const float* deltac;
  float* dKp;           // [B*Hq, npad, D] fp32 per-query-head partial gradients
  float* dVp;
  void* dQ;
  int* sched;           // work list of the dQ items (sched.h)
  size_t order_off;     // where its hand-out order starts
  const int* list;      // [B*Hq, list_stride] the heads' key lists
  int list_stride;
  const int* qvis;      // [B*Hq, N] visible packed keys per kept-query position
  const int* kfirst;    // [B*Hq, npad] first kept-query position that sees a packed key
  int nsplit;           // most workgroups that share the query tiles of one key tile (bf16 key kernel)
  int split_len;        // query tiles per split, at least (bf16: at most, see key_list_block)
  long long plane;      // floats between the partial-gradient planes of two splits
  int* klist;           // work list of the key items (sched.h); null: fp32
  // In-place block lists (TILEMAP kernels): Kn, Vn, Kt hold every KV head once, in token order ([B*Hkv, npad_kv, D]),
  // and tile t of a head's key list is tile tile_map[bh * tile_stride + t] of its KV head's copy.
  const int* tile_map;
  int tile_stride;
  int npad_kv;          // rows per (head) buffer of Kn / Vn / Kt: npad for the gathered copies
};

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int r0) {
  union { bf16x8 v; unsigned u[4]; } o;
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) o.u[jj] = pack_bf16x2(v[r0 + 2 * jj], v[r0 + 2 * jj + 1]);
  return o.v;
}

constexpr int kKeyWaves = 8;
constexpr int kKeyThreads = kKeyWaves * 64;
static_assert(kKeyTile == kKeyWaves * 32, "32 keys per wavefront");
constexpr int kKeySplitLenF32 = 4;           // fp32: query tiles per split, at least (a workgroup owns 32 keys: needed sooner)
constexpr int kKeySplitLen = 128;            // bf16: query tiles per split, at most (64..128 measure alike, 32 and 256 worse)
constexpr int kKeyMaxSplits = 4;             // at most 8: a work item carries the split in 3 bits
// ------------------------------------------------------------------ fp32
//
// Both kernels divide the work as the fp32 forward does: a workgroup owns 32 rows (keys, or kept queries), its
// wavefronts share the 32-row blocks of the other side, every fourth or eighth block each, and add their partial gradients at the
// end in wavefront order.  Operands come straight from memory in the order of the matrix instructions (pack.hip).  Bound
// by the fp32 matrix cores (64 cycles per 32x32x2 step); four times the workgroups and a quarter of the chain of the
// kernels with 128 rows per workgroup and tiles staged without overlap: 161 + 71 us -> 19 + 21 us at 1k tokens, 2 heads,
// d = 64 (of the 19 us, 39 without the splits of the queries).
// Wavefronts per workgroup: as many as its registers allow (d = 64 fits two per SIMD: 36 workgroups of
// four took 44 us in the key kernel where eight took 39).
template <int D>
constexpr int kF32Waves = D == 64 ? 8 : 4;
template <int D>
constexpr int kF32Threads = kF32Waves<D> * 64;

// out[row][d] = scale * sum over the wavefronts of acc (a 32 x D tile held as accumulators: column = row, registers = d)
template <int D, typename Store>
__device__ __forceinline__ void merge_waves(float (*sO)[32][D + 4], const f32x16 (&acc)[D / 32], float scale, Store store) {
  const int lane = lane_id(), wave = threadIdx.x >> 6, ln = lane & 31, h = lane >> 5;
  __syncthreads();
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 v = {acc[db][q4 * 4], acc[db][q4 * 4 + 1], acc[db][q4 * 4 + 2], acc[db][q4 * 4 + 3]};
      *reinterpret_cast<f32x4*>(&sO[wave][ln][db * 32 + 8 * q4 + 4 * h]) = v;
    }
  __syncthreads();
#pragma unroll
  for (int c = threadIdx.x; c < 32 * (D / 4); c += kF32Threads<D>) {
    const int row = c / (D / 4), d = c % (D / 4) * 4;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kF32Waves<D>; ++w) x += *reinterpret_cast<const f32x4*>(&sO[w][row][d]);
    store(row, d, x * scale);
  }
}

// One 32-row block in fragment order (A or B operand of a product that contracts over d) / in k-packed order (A operand of
// a product that contracts over the rows).
template <int D>
__device__ __forceinline__ void load_frag(f32x4 (&f)[D / 8], const float* block) {
#pragma unroll
  for (int ks = 0; ks < D / 8; ++ks) f[ks] = *reinterpret_cast<const f32x4*>(block + (ks * 64 + lane_id()) * 4);
}
template <int D>
__device__ __forceinline__ void load_packed(f32x4 (&f)[4][D / 32], const float* block) {
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
      f[q4][db] = *reinterpret_cast<const f32x4*>(block + ((q4 * (D / 32) + db) * 64 + lane_id()) * 4);
}
template <int D>
__device__ __forceinline__ f32x16 product_d(const f32x4 (&a)[D / 8], const f32x4 (&b)[D / 8]) {
  f32x16 s;
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 8; ++ks)
#pragma unroll
    for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ks][e], b[ks][e], s, 0, 0, 0);
  return s;
}
template <int D>
__device__ __forceinline__ void add_product_rows(f32x16 (&acc)[D / 32], const f32x4 (&a)[4][D / 32], const f32x16& x) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
      acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[r >> 2][db][r & 3], x[r], acc[db], 0, 0, 0);
}

// Block `block` of npad / 32 * nsplit * B*Hq, heads fastest; the first keys, which the most queries see, first.  dK', dV' of 32
// listed keys, or of the share of the queries that a split of their 256-key tile takes (as in the bf16 kernel).
template <int D>
__device__ __forceinline__ void key_f32_block(const BwdParams& p, int block, float (*sO)[32][D + 4]) {
  constexpr int NB = D / 32;
  const Layer& L = p.L;
  const int BH = L.B * L.Hq, bh = block % BH, sp = block / BH % p.nsplit, b = bh / L.Hq;
  const int slot0 = block / BH / p.nsplit * 32;
  const int nkeys = min(p.budget[budget_slot(L.bph, b, bh)], p.b_cap);
  if (slot0 >= nkeys) return;
  const int nq = p.q_cnt[bh];
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const int* kfirst = p.kfirst + (long long)bh * p.npad;
  const int my_first = kfirst[slot0 + ln] - 4 * h;          // query positions below it do not see this lane's key
  const int q_first = kfirst[slot0 / kKeyTile * kKeyTile] / kKeyQ, n_all = cdiv(nq, kKeyQ) - q_first;
  const int n_sp = key_tile_splits(n_all, p.nsplit, p.split_len), per_split = cdiv(n_all, n_sp) * kKeyQ;
  if (sp >= n_sp) return;
  const int q_begin = max(kfirst[slot0], q_first * kKeyQ + sp * per_split) / 32;
  const int q_end = min(nq, q_first * kKeyQ + (sp + 1) * per_split);
  const long long kv = ((long long)bh * p.npad + slot0) * D, qo = (long long)bh * p.nqpad;
  f32x4 kf[D / 8], vf[D / 8];
  load_frag<D>(kf, static_cast<const float*>(p.Kn) + kv);
  load_frag<D>(vf, static_cast<const float*>(p.Vn) + kv);
  f32x16 dk[NB], dv[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[db][r] = 0.f, dv[db][r] = 0.f;
  for (int t = q_begin + wave; t * 32 < q_end; t += kF32Waves<D>) {
    const long long row = (qo + t * 32) * D;
    f32x4 qa[D / 8], ga[D / 8], qt[4][NB], gt[4][NB], lse[4], del[4];
    load_frag<D>(qa, static_cast<const float*>(p.Qn) + row);
    load_frag<D>(ga, static_cast<const float*>(p.dOn) + row);
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      lse[q4] = *reinterpret_cast<const f32x4*>(p.lse2c + qo + t * 32 + 8 * q4 + 4 * h);
      del[q4] = *reinterpret_cast<const f32x4*>(p.deltac + qo + t * 32 + 8 * q4 + 4 * h);
    }
    load_packed<D>(qt, static_cast<const float*>(p.Qt) + row);
    load_packed<D>(gt, static_cast<const float*>(p.dOt) + row);
    f32x16 s = product_d<D>(qa, kf), dp = product_d<D>(ga, vf);      // rows: queries 8 (r / 4) + 4 h + r % 4
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pv = fast_exp2(fmaf(s[r], c2, -lse[r >> 2][r & 3]));
      if (t * 32 + 8 * (r >> 2) + (r & 3) < my_first) pv = 0.f;
      s[r] = pv;
      dp[r] = pv * (dp[r] - del[r >> 2][r & 3]);
    }
    add_product_rows<D>(dv, gt, s);
    add_product_rows<D>(dk, qt, dp);
  }
  float *dkp = p.dKp + sp * p.plane + kv, *dvp = p.dVp + sp * p.plane + kv;
  merge_waves<D>(sO, dk, L.scale, [&](int row, int d, const f32x4& x) { *reinterpret_cast<f32x4*>(dkp + row * D + d) = x; });
  merge_waves<D>(sO, dv, 1.f, [&](int row, int d, const f32x4& x) { *reinterpret_cast<f32x4*>(dvp + row * D + d) = x; });
}

// Block `block` of cdiv(N, 32) * B*Hq, heads fastest; a head's last rows, which see the most keys, first.  dQ of 32 kept queries.
template <int D>
__device__ __forceinline__ void dq_f32_block(const BwdParams& p, int block, float (*sO)[32][D + 4]) {
  constexpr int NB = D / 32;
  const Layer& L = p.L;
  const int BH = L.B * L.Hq, bh = block % BH, b = bh / L.Hq, i = bh % L.Hq;
  const int nq = p.q_cnt[bh];
  const int tq = cdiv(nq, 32) - 1 - block / BH;
  if (tq < 0) return;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const int* qlist = p.q_idx + (long long)bh * L.N;
  const int* qvis = p.qvis + (long long)bh * L.N;
  const long long qo = (long long)bh * p.nqpad + tq * 32;
  const int pos_c = min(tq * 32 + ln, nq - 1);
  const int qvisible = qvis[pos_c] - 4 * h, nblocks = cdiv(qvis[min(tq * 32 + 31, nq - 1)], 32);
  const float lse = p.lse2c[qo + ln], delta = p.deltac[qo + ln];
  f32x4 qf[D / 8], gf[D / 8];
  load_frag<D>(qf, static_cast<const float*>(p.Qn) + qo * D);
  load_frag<D>(gf, static_cast<const float*>(p.dOn) + qo * D);
  f32x16 dq[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[db][r] = 0.f;
  for (int t = wave; t < nblocks; t += kF32Waves<D>) {
    const long long kv = ((long long)bh * p.npad + t * 32) * D;
    f32x4 kf[D / 8], vf[D / 8], kt[4][NB];
    load_frag<D>(kf, static_cast<const float*>(p.Kn) + kv);
    load_frag<D>(vf, static_cast<const float*>(p.Vn) + kv);
    load_packed<D>(kt, static_cast<const float*>(p.Kt) + kv);
    f32x16 s = product_d<D>(kf, qf), dp = product_d<D>(vf, gf);      // rows: keys 8 (r / 4) + 4 h + r % 4
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pv = fast_exp2(fmaf(s[r], c2, -lse));
      if (t * 32 + 8 * (r >> 2) + (r & 3) >= qvisible) pv = 0.f;
      dp[r] = pv * (dp[r] - delta);
    }
    add_product_rows<D>(dq, kt, dp);
  }
  float* head = static_cast<float*>(p.dQ) + b * L.qs[0] + i * L.qs[1];
  merge_waves<D>(sO, dq, L.scale, [&](int row, int d, const f32x4& x) {
    if (tq * 32 + row < nq) *reinterpret_cast<f32x4*>(head + (long long)qlist[tq * 32 + row] * L.qs[2] + d) = x;
  });
}

// Both in one launch, key blocks first: neither fills the chip on the sequences that come here (1024 tokens, 2 heads, d = 64: 19
// and 20 us one after the other), and neither needs the other.
template <int D>
__global__ __launch_bounds__(kF32Threads<D>, 1) void attn_bwd_f32_kernel(BwdParams p, int key_blocks) {
  __shared__ __attribute__((aligned(16))) float sO[kF32Waves<D>][32][D + 4];
  if ((int)blockIdx.x < key_blocks) return key_f32_block<D>(p, blockIdx.x, sO);
  dq_f32_block<D>(p, (int)blockIdx.x - key_blocks, sO);
}

// fp32, long sequences (f32_short): workgroups of 128 keys, or of 128 kept queries from the work list, 32 per wavefront;
// tiles of 64 rows of the other side staged row by row through LDS, Q and dO straight from the caller's arrays.  One plane
// of dK', dV', no other copies than K and V: a quarter of the scratch.
constexpr int kF32Keys = 128;

// grid: (npad / 128, B*Hq)
template <int D>
__global__ __launch_bounds__(kThreads, 1) void attn_bwd_key_f32_long_kernel(BwdParams p) {
  constexpr int LD = D + 8;                                 // row pitch of the tiles
  constexpr int CPR = D / 4, kChunks = kKeyQ * CPR / kThreads;
  __shared__ __attribute__((aligned(16))) float sq[kKeyQ * LD], sg[kKeyQ * LD];
  __shared__ __attribute__((aligned(16))) float sLse[kKeyQ], sDel[kKeyQ];
  const Layer& L = p.L;
  const int slot0 = blockIdx.x * kF32Keys, bh = blockIdx.y, b = bh / L.Hq, i = bh % L.Hq;
  const int nkeys = min(p.budget[budget_slot(L.bph, b, bh)], p.b_cap);
  if (slot0 >= nkeys) return;
  const int nq = p.q_cnt[bh];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int ln = lane & 31, h = lane >> 5;
  const int slot = slot0 + wave * 32 + ln;                  // this lane's key slot (< npad by construction)
  const float c2 = L.scale * kLog2e;
  const int* qlist = p.q_idx + (long long)bh * L.N;
  const int* kfirst = p.kfirst + (long long)bh * p.npad;
  const int my_first = kfirst[slot] - 4 * h;                // query positions below it do not see this lane's key
  const bool has_pad = slot0 + kF32Keys > nkeys;
  const int q_full_pos = has_pad ? 0x7fffffff : kfirst[slot0 + kF32Keys - 1];    // tiles from this position on need no mask
  const int n_qtiles = cdiv(nq, kKeyQ);
  f32x4 kf[D / 8], vf[D / 8];                               // resident: B operands, lane = key column
  const long long kv = ((long long)bh * p.npad + slot) * D;
#pragma unroll
  for (int ks = 0; ks < D / 8; ++ks) {
    kf[ks] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.Kn) + kv + ks * 8 + h * 4);
    vf[ks] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.Vn) + kv + ks * 8 + h * 4);
  }
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[db][r] = 0.f, dv[db][r] = 0.f;
  const float* qbase = static_cast<const float*>(p.Q) + b * L.qs[0] + i * L.qs[1];
  const float* gbase = static_cast<const float*>(p.dO) + b * L.qs[0] + i * L.qs[1];
  for (int t = kfirst[slot0] / kKeyQ; t < n_qtiles; ++t) {
    const int pos0 = t * kKeyQ;
    __syncthreads();
    u32x4 stQ[kChunks], stG[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int ch = threadIdx.x + c * kThreads, col = ch % CPR * 4, pos = pos0 + ch / CPR;
      stQ[c] = stG[c] = u32x4{0u, 0u, 0u, 0u};
      if (pos < nq) {
        const long long at = (long long)qlist[pos] * L.qs[2] + col;
        stQ[c] = *reinterpret_cast<const u32x4*>(qbase + at);
        stG[c] = *reinterpret_cast<const u32x4*>(gbase + at);
      }
    }
    float stL = 0.f, stD = 0.f;
    if (threadIdx.x < kKeyQ) {
      stL = p.lse2c[(long long)bh * p.nqpad + pos0 + threadIdx.x];
      stD = p.deltac[(long long)bh * p.nqpad + pos0 + threadIdx.x];
    }
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int ch = threadIdx.x + c * kThreads, at = ch / CPR * LD + ch % CPR * 4;
      *reinterpret_cast<u32x4*>(sq + at) = stQ[c];
      *reinterpret_cast<u32x4*>(sg + at) = stG[c];
    }
    if (threadIdx.x < kKeyQ) {
      sLse[threadIdx.x] = stL;
      sDel[threadIdx.x] = stD;
    }
    __syncthreads();
    const bool masked = pos0 < q_full_pos;
#pragma unroll
    for (int qb = 0; qb < kKeyQ / 32; ++qb) {
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f, dp[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < D / 8; ++ks) {
        const f32x4 qa = *reinterpret_cast<const f32x4*>(sq + (qb * 32 + ln) * LD + ks * 8 + h * 4);
        const f32x4 ga = *reinterpret_cast<const f32x4*>(sg + (qb * 32 + ln) * LD + ks * 8 + h * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = __builtin_amdgcn_mfma_f32_32x32x2f32(qa[e], kf[ks][e], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x2f32(ga[e], vf[ks][e], dp, 0, 0, 0);
        }
      }
      // accumulator rows are queries 8 (r/4) + 4 h + r%4 of this block, the column is this lane's key
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int qo = qb * 32 + 8 * q4 + 4 * h;
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(&sLse[qo]), d4 = *reinterpret_cast<const f32x4*>(&sDel[qo]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = q4 * 4 + e;
          float pv = fast_exp2(fmaf(s[r], c2, -l4[e]));
          if (masked && pos0 + qb * 32 + 8 * q4 + e < my_first) pv = 0.f;
          s[r] = pv;
          dp[r] = pv * (dp[r] - d4[e]);
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int qrow = qb * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
          dv[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(sg[qrow * LD + db * 32 + ln], s[r], dv[db], 0, 0, 0);
          dk[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(sq[qrow * LD + db * 32 + ln], dp[r], dk[db], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const long long at = kv + db * 32 + 8 * q4 + 4 * h;
      const f32x4 x = {dk[db][q4 * 4], dk[db][q4 * 4 + 1], dk[db][q4 * 4 + 2], dk[db][q4 * 4 + 3]};
      const f32x4 y = {dv[db][q4 * 4], dv[db][q4 * 4 + 1], dv[db][q4 * 4 + 2], dv[db][q4 * 4 + 3]};
      *reinterpret_cast<f32x4*>(p.dKp + at) = x * L.scale;
      *reinterpret_cast<f32x4*>(p.dVp + at) = y;
    }
}

template <int D>
__global__ __launch_bounds__(kThreads, 1) void attn_bwd_dq_f32_long_kernel(BwdParams p) {
  constexpr int LD = D + 8;
  constexpr int CPR = D / 4, kChunks = kTileN * CPR / kThreads;
  __shared__ __attribute__((aligned(16))) float sk[kTileN * LD], sv[kTileN * LD];
  __shared__ int sItem;
  const Layer& L = p.L;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  for (;;) {                                 // persistent: one (head, query tile) per iteration
    __syncthreads();
    if (threadIdx.x == 0) sItem = sched_next(p.sched, 1);
    __syncthreads();
    const int item = sItem;
    if (item < 0) break;
    int bh, tq;
    sched_decode(p.sched, p.order_off, item, bh, tq);
    const int b = bh / L.Hq, i = bh % L.Hq, nq = p.q_cnt[bh];
    const int* qlist = p.q_idx + (long long)bh * L.N;
    const int* qvis = p.qvis + (long long)bh * L.N;
    const int pos_first = tq * kTileM, pos_last = min(pos_first + kTileM, nq) - 1;
    const int n_full_tiles = qvis[pos_first] / kTileN, ntiles = cdiv(qvis[pos_last], kTileN);
    const int qpos = pos_first + wave * 32 + ln, qpos_c = min(qpos, nq - 1), qvisible = qvis[qpos_c] - 4 * h;
    const float lse2 = p.lse2c[(long long)bh * p.nqpad + qpos_c], delta = p.deltac[(long long)bh * p.nqpad + qpos_c];
    const long long row_off = b * L.qs[0] + i * L.qs[1] + (long long)qlist[qpos_c] * L.qs[2];
    f32x4 qf[D / 8], gf[D / 8];
#pragma unroll
    for (int ks = 0; ks < D / 8; ++ks) {
      qf[ks] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.Q) + row_off + ks * 8 + h * 4);
      gf[ks] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.dO) + row_off + ks * 8 + h * 4);
    }
    f32x16 dq[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[db][r] = 0.f;
    const float* kn = static_cast<const float*>(p.Kn) + (long long)bh * p.npad * D;
    const float* vn = static_cast<const float*>(p.Vn) + (long long)bh * p.npad * D;
    for (int t = 0; t < ntiles; ++t) {
      __syncthreads();
      u32x4 stK[kChunks], stV[kChunks];
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const long long at = (long long)t * kTileN * D + (threadIdx.x + c * kThreads) * 4;
        stK[c] = *reinterpret_cast<const u32x4*>(kn + at);
        stV[c] = *reinterpret_cast<const u32x4*>(vn + at);
      }
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const int ch = threadIdx.x + c * kThreads, at = ch / CPR * LD + ch % CPR * 4;
        *reinterpret_cast<u32x4*>(sk + at) = stK[c];
        *reinterpret_cast<u32x4*>(sv + at) = stV[c];
      }
      __syncthreads();
      f32x16 s[2], dp[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f, dp[kb][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 8; ++ks) {
          const f32x4 ka = *reinterpret_cast<const f32x4*>(sk + (kb * 32 + ln) * LD + ks * 8 + h * 4);
          const f32x4 va = *reinterpret_cast<const f32x4*>(sv + (kb * 32 + ln) * LD + ks * 8 + h * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[e], qf[ks][e], s[kb], 0, 0, 0);
            dp[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[e], gf[ks][e], dp[kb], 0, 0, 0);
          }
        }
      }
      const bool masked = t >= n_full_tiles;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float pv = fast_exp2(fmaf(s[kb][r], c2, -lse2));
          if (masked && t * kTileN + kb * 32 + 8 * (r >> 2) + (r & 3) >= qvisible) pv = 0.f;
          dp[kb][r] = pv * (dp[kb][r] - delta);
        }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int slot = kb * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
#pragma unroll
          for (int db = 0; db < D / 32; ++db)
            dq[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(sk[slot * LD + db * 32 + ln], dp[kb][r], dq[db], 0, 0, 0);
        }
    }
    if (qpos < nq) {
      float* out = static_cast<float*>(p.dQ) + row_off;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x4 x = {dq[db][q4 * 4], dq[db][q4 * 4 + 1], dq[db][q4 * 4 + 2], dq[db][q4 * 4 + 3]};
          *reinterpret_cast<f32x4*>(out + db * 32 + 8 * q4 + 4 * h) = x * L.scale;
        }
    }
  }
}

// ------------------------------------------------------------------ dQ, bf16 fast path
//
// Same organisation as the bf16 forward kernel: 512 threads = 8 wavefronts x 32 kept queries (256-row work
// items from the longest-first persistent list), K / V / K^T tiles of 64 keys streamed memory -> LDS with
// LDS-DMA loads into a ring of kDqStages buffers in fragment order, one
// barrier per tile, the loads of tile t+2 spread over the MFMAs of tile t, causal mask from the per-query
// visible-prefix count.  Per tile and wavefront: S^T = K Q^T and dP^T = V dO^T (32 MFMAs), dS^T on the
// vector ALU, dQ^T += K^T dS^T (16 MFMAs).

constexpr int kDqWaves = 8;
constexpr int kDqThreads = kDqWaves * 64;
constexpr int kDqTileM = kDqWaves * 32;
constexpr int kDqStages = 3;

constexpr int kBwdMaxMapTiles = 2048;               // key tiles of one head in the in-place variant (128k tokens)

template <int D>
constexpr int kDqLds = kDqStages * 3 * kTileN * D * 2;
template <int D, bool TILEMAP>
__device__ __forceinline__ void dq_items(const BwdParams& p, unsigned char* smem, int4& sItem, int* sTileMap) {
  typedef u16 T;
  constexpr int kOpBytes = kTileN * D * 2;           // one operand tile
  constexpr int kStageBytes = 3 * kOpBytes;          // K, V, K k-packed
  constexpr int LPH = kOpBytes / 1024 / kDqWaves;    // load instructions per operand per wavefront per tile
  constexpr int LPT = 3 * LPH;
  constexpr int NB = D / 32;
  static_assert(LPH >= 1, "tile too small for the copy scheme");
  static_assert(kDqLds<D> == kDqStages * kStageBytes, "");

  const Layer& L = p.L;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int lane_b = lane * 16;                      // copies and fragment reads: 16 bytes a lane, in lane order

  const int n_items = p.sched[kSchedTotal];          // one queue, longest item first
  for (;;) {
  __syncthreads();
  if (threadIdx.x == 0) {
    int bh = -1, tq = 0, full = 0, all = 0;
    const int k = atomicAdd(p.sched + kSchedCursor, 1);
    if (k < n_items) {
      sched_decode(p.sched, p.order_off, k, bh, tq);
      const int* qvis = p.qvis + (long long)bh * L.N;
      full = qvis[tq * kDqTileM];
      all = qvis[min((tq + 1) * kDqTileM, p.q_cnt[bh]) - 1];
    }
    sItem = make_int4(bh, tq, full, all);
  }
  __syncthreads();
  const int bh = __builtin_amdgcn_readfirstlane(sItem.x);   // wave-uniform, and known to be: tile bases stay in SGPRs
  const int tq = __builtin_amdgcn_readfirstlane(sItem.y);
  if (bh < 0) break;
  const int b = bh / L.Hq, i = bh % L.Hq;
  const int nq = p.q_cnt[bh];
  const int* qlist = p.q_idx + (long long)bh * L.N;
  const int* qvis = p.qvis + (long long)bh * L.N;
  const int pos_first = tq * kDqTileM;
  const int n_full_tiles = __builtin_amdgcn_readfirstlane(sItem.z) / kTileN;
  const int ntiles = cdiv(__builtin_amdgcn_readfirstlane(sItem.w), kTileN);
  if constexpr (TILEMAP) {                                   // this item's share of the head's tile map
    const int* tm = p.tile_map + (long long)bh * p.tile_stride;
    for (int t = threadIdx.x; t < ntiles; t += kDqThreads) sTileMap[t] = tm[t];
    __syncthreads();
  }

  const int qpos = pos_first + wave * 32 + ln;
  const bool qvalid = qpos < nq;
  const int qpos_c = min(qpos, nq - 1);
  const int qrow = qlist[qpos_c];
  const int qvisible = qvis[qpos_c] - 4 * h;
  // the packed rows: no list entry between the item and the loads (rows past the last are garbage that nobody stores)
  const long long packed = (long long)bh * p.nqpad + min(pos_first + wave * 32, (nq - 1) & ~31);
  const float lse2 = p.lse2c[(long long)bh * p.nqpad + qpos_c];
  const float delta = p.deltac[(long long)bh * p.nqpad + qpos_c];
  const T* qptr = static_cast<const T*>(p.Qn) + packed * D + lane * 8;
  const T* gptr = static_cast<const T*>(p.dOn) + packed * D + lane * 8;
  bf16x8 qf[D / 16], gf[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    qf[ks] = *reinterpret_cast<const bf16x8*>(qptr + ks * 512);
    gf[ks] = *reinterpret_cast<const bf16x8*>(gptr + ks * 512);
  }
  float lse2r = lse2, deltar = delta;
  // finish every ordinary load here: a compiler-placed wait inside the tile loop would drain the ring
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    asm volatile("" : "+v"(qf[ks]));
    asm volatile("" : "+v"(gf[ks]));
  }
  asm volatile("" : "+v"(lse2r), "+v"(deltar));

  f32x16 dq[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[db][r] = 0.f;

  const int bhx = TILEMAP ? b * L.Hkv + i / L.G : bh;
  const T* kn = static_cast<const T*>(p.Kn) + (long long)bhx * p.npad_kv * D;
  const T* vn = static_cast<const T*>(p.Vn) + (long long)bhx * p.npad_kv * D;
  const T* kt = static_cast<const T*>(p.Kt) + (long long)bhx * p.npad_kv * D;
  auto issue_part = [&](int t, int part) {
    const int op = part / LPH, j = part % LPH;
    const int at = j * kDqWaves + wave;
    const unsigned dst = lds_base + (unsigned)(t % kDqStages) * kStageBytes + op * kOpBytes + at * 1024;
    // where tile t of the key list lives (wave-uniform: the tile base stays in scalar registers)
    const int src = TILEMAP ? __builtin_amdgcn_readfirstlane(sTileMap[t]) : t;
    gload_lds16((op == 0 ? kn : op == 1 ? vn : kt) + (long long)src * kTileN * D + at * 512, lane_b, dst);
  };
  auto issue_tile = [&](int t) {
#pragma unroll
    for (int j = 0; j < LPT; ++j) issue_part(t, j);
  };

  constexpr int NA = 4 * (D / 16);           // MFMAs of the S^T and dP^T tiles: 2 key blocks x D/16 k-steps x 2
  constexpr int NC = 4 * NB;                 // MFMAs of the dQ^T update: 4 key steps x D/32 row blocks
  constexpr int kAhead = 2;
  static_assert(NA % (2 * LPH) == 0 && NC % LPH == 0, "loads are spread evenly over the MFMAs");
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  auto compute_tile = [&](int t, int pre, bool masked) {
    const unsigned char* st = smem + (t % kDqStages) * kStageBytes;
    // chunk c of phase A: key block kb, k-step ks, operand (0: K for S, 1: V for dP)
    auto afrag = [&](int c) {
      const int which = c % 2, ks = (c / 2) % (D / 16), kb = c / (D / 8);
      return *reinterpret_cast<const bf16x8*>(st + lane_b + which * kOpBytes + (kb * (D / 16) + ks) * 1024);
    };
    auto cfrag = [&](int c) {
      return *reinterpret_cast<const bf16x8*>(st + lane_b + 2 * kOpBytes + c * 1024);
    };
    f32x16 s[2], dp[2];
    bf16x8 fa[kAhead];
#pragma unroll
    for (int c = 0; c < kAhead; ++c) fa[c] = afrag(c);
#pragma unroll
    for (int c = 0; c < NA; ++c) {
      const int which = c % 2, ks = (c / 2) % (D / 16), kb = c / (D / 8);
      __builtin_amdgcn_sched_barrier(0);
      if (which == 0) s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c % kAhead], qf[ks], ks == 0 ? zero16 : s[kb], 0, 0, 0);
      else dp[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c % kAhead], gf[ks], ks == 0 ? zero16 : dp[kb], 0, 0, 0);
      if (c + kAhead < NA) fa[c % kAhead] = afrag(c + kAhead);
      if (c % (NA / (2 * LPH)) == 0 && pre >= 0) issue_part(pre, c / (NA / (2 * LPH)));      // K and V parts of tile t+2
    }
    __builtin_amdgcn_sched_barrier(0);
    // dS^T = P^T (dP^T - delta); the lane's query fixes lse and delta, the register fixes the key.  Only the tiles
    // at the causal diagonal of the item pay for the position compares (a wavefront-uniform branch).
    bf16x8 fc[kAhead];
#pragma unroll
    for (int c = 0; c < kAhead; ++c) fc[c] = cfrag(c);
    bf16x8 dsf[4];
    auto weights = [&](auto with_mask) {
      const int rel = qvisible - t * kTileN;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float pv = fast_exp2(fmaf(s[kb][r], c2, -lse2r));
          if (decltype(with_mask)::value && kb * 32 + 8 * (r >> 2) + (r & 3) >= rel) pv = 0.f;
          dp[kb][r] = pv * (dp[kb][r] - deltar);
        }
        dsf[kb * 2] = pack8(dp[kb], 0);
        dsf[kb * 2 + 1] = pack8(dp[kb], 8);
      }
    };
    if (masked) weights(std::true_type{});
    else weights(std::false_type{});
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int t16 = c / NB, db = c % NB;
      __builtin_amdgcn_sched_barrier(0);
      dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[c % kAhead], dsf[t16], dq[db], 0, 0, 0);
      if (c + kAhead < NC) fc[c % kAhead] = cfrag(c + kAhead);
      if (c % (NC / LPH) == 0 && pre >= 0) issue_part(pre, 2 * LPH + c / (NC / LPH));            // K^T parts
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // Ring of kDqStages buffers, one barrier per tile: at the top of step t the tiles up to t+1 have been
  // issued; after its barrier everyone is done with tile t-1, whose buffer takes tile t+2.
  static_assert(kDqStages == 3, "the wait counts assume this ring depth");
  if (ntiles > 0) {
    wait_vmcnt<0>();
    issue_tile(0);
    if (ntiles > 1) issue_tile(1);
    for (int t = 0; t < ntiles; ++t) {
      if (t + 1 < ntiles) wait_vmcnt<LPT>();
      else wait_vmcnt<0>();
      __syncthreads();
      compute_tile(t, t + 2 < ntiles ? t + 2 : -1, t >= n_full_tiles);
    }
  }

  if (qvalid) {
    T* optr = static_cast<T*>(p.dQ) + b * L.qs[0] + i * L.qs[1] + (long long)qrow * L.qs[2];
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d = db * 32 + 8 * q4 + 4 * h;
        uint2 w;
        w.x = pack_bf16x2(dq[db][q4 * 4 + 0] * L.scale, dq[db][q4 * 4 + 1] * L.scale);
        w.y = pack_bf16x2(dq[db][q4 * 4 + 2] * L.scale, dq[db][q4 * 4 + 3] * L.scale);
        *reinterpret_cast<uint2*>(optr + d) = w;
      }
  }
  }  // work-item loop
}

// ------------------------------------------------------------------ dQ, bf16, few rows
//
// Items of 32 kept queries whose eight wavefronts share the 32-key blocks of the head's list, operands straight from memory in
// fragment order, partial sums added in wavefront order; no work list.  A 256-row item walks its tiles one after the other at 1.5
// to 2 us each, and where the heads are few there is nothing else to do meanwhile (one head of 8192 tokens: 32 items of up to 128
// tiles on 256 CUs).  Bound by the loads: every item fetches its head's K, V and K^T, eight times what a 256-row item does, from
// the caches; hence the line (bwd_few_rows).
template <int D>
constexpr int kDqRowsLds = 2 * 32 * D * 2 + kKeyWaves * 32 * (D + 4) * 4;
template <int D, bool TILEMAP>
__device__ __forceinline__ void dq_row_items(const BwdParams& p, unsigned char* smem, int4& sItem) {
  typedef u16 T;
  constexpr int KS = D / 16, NB = D / 32, kOp = 32 * D * 2;
  unsigned char *sQ = smem, *sG = smem + kOp;
  float (*sO)[32][D + 4] = reinterpret_cast<float (*)[32][D + 4]>(smem + 2 * kOp);
  const Layer& L = p.L;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const int BH = L.B * L.Hq, n_slots = cdiv(L.N, 32) * BH;         // heads fastest; a head's last rows, which see the most keys, first
  for (;;) {
    __syncthreads();                           // LDS of the item before is no longer read
    if (threadIdx.x == 0) {
      int bh = -1, tq = -1;
      for (int k = atomicAdd(&p.klist[kKeyListRows], 1); k < n_slots; k = atomicAdd(&p.klist[kKeyListRows], 1)) {
        tq = cdiv(p.q_cnt[k % BH], 32) - 1 - k / BH;
        if (tq >= 0) {
          bh = k % BH;
          break;
        }
      }
      sItem = make_int4(bh, tq, 0, 0);
    }
    __syncthreads();
    const int bh = __builtin_amdgcn_readfirstlane(sItem.x), tq = __builtin_amdgcn_readfirstlane(sItem.y);
    if (bh < 0) break;
    const int b = bh / L.Hq, i = bh % L.Hq, nq = p.q_cnt[bh];
    const int* qlist = p.q_idx + (long long)bh * L.N;
    const int* qvis = p.qvis + (long long)bh * L.N;
    const long long qo = (long long)bh * p.nqpad + tq * 32;
    const int qvisible = qvis[min(tq * 32 + ln, nq - 1)] - 4 * h;
    const int n_full = qvis[tq * 32] / 32, nblocks = cdiv(qvis[min(tq * 32 + 31, nq - 1)], 32);
    const float lse = p.lse2c[qo + ln], delta = p.deltac[qo + ln];
    if (threadIdx.x < kOp / 16) {
      *reinterpret_cast<u32x4*>(sQ + threadIdx.x * 16) = *reinterpret_cast<const u32x4*>(static_cast<const T*>(p.Qn) + qo * D + threadIdx.x * 8);
      *reinterpret_cast<u32x4*>(sG + threadIdx.x * 16) = *reinterpret_cast<const u32x4*>(static_cast<const T*>(p.dOn) + qo * D + threadIdx.x * 8);
    }
    const int bhx = TILEMAP ? b * L.Hkv + i / L.G : bh;
    const long long head = (long long)bhx * p.npad_kv * D + lane * 8;
    const T *kn = static_cast<const T*>(p.Kn) + head, *vn = static_cast<const T*>(p.Vn) + head, *kt = static_cast<const T*>(p.Kt) + head;
    auto block_off = [&](int t) {
      if (!TILEMAP) return (long long)t * 32 * D;
      return (long long)(__builtin_amdgcn_readfirstlane(p.tile_map[(long long)bh * p.tile_stride + t / 2]) * 2 + t % 2) * 32 * D;
    };
    bf16x8 kf[KS], vf[KS];
    auto load_kv = [&](int t) {
      const long long o = block_off(t);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        kf[ks] = *reinterpret_cast<const bf16x8*>(kn + o + ks * 512);
        vf[ks] = *reinterpret_cast<const bf16x8*>(vn + o + ks * 512);
      }
    };
    f32x16 dq[NB];
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[db][r] = 0.f;
    if (wave < nblocks) load_kv(wave);
    __syncthreads();
    for (int t = wave; t < nblocks; t += kKeyWaves) {
      bf16x8 ktf[2][NB];
      const T* ktb = kt + block_off(t);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int db = 0; db < NB; ++db) ktf[u][db] = *reinterpret_cast<const bf16x8*>(ktb + (u * NB + db) * 512);
      const unsigned char* frag = sQ + loop_lane() * 16;          // anew: resident, the fragments would take 64 registers
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f, dp[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], *reinterpret_cast<const bf16x8*>(frag + ks * 1024), s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks], *reinterpret_cast<const bf16x8*>(frag + kOp + ks * 1024), dp, 0, 0, 0);
      }
      if (t + kKeyWaves < nblocks) load_kv(t + kKeyWaves);
      const bool masked = t >= n_full;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float pv = fast_exp2(fmaf(s[r], c2, -lse));
        if (masked && t * 32 + 8 * (r >> 2) + (r & 3) >= qvisible) pv = 0.f;
        dp[r] = pv * (dp[r] - delta);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8 ds = pack8(dp, u * 8);
#pragma unroll
        for (int db = 0; db < NB; ++db) dq[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf[u][db], ds, dq[db], 0, 0, 0);
      }
    }
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4 v = {dq[db][q4 * 4], dq[db][q4 * 4 + 1], dq[db][q4 * 4 + 2], dq[db][q4 * 4 + 3]};
        *reinterpret_cast<f32x4*>(&sO[wave][ln][db * 32 + 8 * q4 + 4 * h]) = v;
      }
    __syncthreads();
    const int row = threadIdx.x / (D / 8), d = threadIdx.x % (D / 8) * 8;      // a thread adds eight of d
    if (row < 32 && tq * 32 + row < nq) {
      f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
#pragma unroll
      for (int w = 0; w < kKeyWaves; ++w) {
        x += *reinterpret_cast<const f32x4*>(&sO[w][row][d]);
        y += *reinterpret_cast<const f32x4*>(&sO[w][row][d + 4]);
      }
      x *= L.scale;
      y *= L.scale;
      T* out = static_cast<T*>(p.dQ) + b * L.qs[0] + i * L.qs[1] + (long long)qlist[tq * 32 + row] * L.qs[2] + d;
      *reinterpret_cast<u32x4*>(out) = u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    }
  }
}

// ------------------------------------------------------------------ dK' and dV', bf16 fast path
//
// The dQ items with the roles of keys and queries swapped: a workgroup of 8 wavefronts owns 256 packed keys of one
// query head (32 per wavefront, K and V fragments resident in registers) and streams tiles of the packed kept rows
// memory -> LDS with LDS-DMA loads into a ring of four: Q and dO in fragment order (operands of S and dP) and k-packed (of the
// updates), 8 KB each, so that a wavefront issues one load per operand and tile, three tiles ahead.  Per 32 queries and
// wavefront: S (D/16 matrix instructions), dP with the weights P of S on the vector ALU under it, dV' += P^T dO with dS
// under it, dK' += dS^T Q.  At d = 128 the fragments (64 registers), the two accumulators (128), S and dP (32), P
// packed and the operands in flight leave a handful of the 256 registers of two wavefronts per SIMD for everything else, so
// all operands lie in lane order (one address for a tile's fragments), what depends on the lane is formed anew per tile
// (loop_lane), and tiles at the causal diagonal have a loop of their own instead of a branch.  A single register that the
// tile loop reloads from scratch costs a tenth of the kernel, because its wait drains the loads in flight: 3084 -> 2750 us at
// 32k, 28 heads.  Tiles of 32 queries, because a stage of 64 would leave the ring two stages.
// Bound: matrix cores, waiting in part for their wavefronts.  dK' and dV' as two kernels, each with an S of its own (5
// products where 4 are needed, Q read twice), took 2226 + 1384 us at 32k, 28 heads, d = 128, this one 2660 to 2750: forward
// and backward there 7500 -> 6541 us, two clips of 3101 at d = 64 214 -> 178 us, blocks at 16k 3540 -> 3044 us (the packs,
// faster too, are a fifth of that), with the same results to the last bit.
// lse * log2e and delta of the tile's queries come with the tile (LDS-DMA of 4 bytes per lane); the causal
// mask is a comparison of the query position with the first position that sees the lane's key.

template <int D>
constexpr int kKeyLds = 4 * (4 * 8192 + 4096 / D / 32 * 256);
template <int D, bool TILEMAP>
__device__ __forceinline__ void key_items(const BwdParams& p, unsigned char* smem, int4& sItem, int* sFirst) {
  typedef u16 T;
  constexpr int CH = D / 8;
  constexpr int NB = D / 32;
  constexpr int KS = D / 16;
  constexpr int kRows = 4096 / D;                    // queries per streamed tile: 8 KB an operand, one load a wavefront
  constexpr int kStages = 4;
  constexpr int kAheadTiles = kStages - 1;
  constexpr int NSMALL = kRows / 32;                 // wavefronts that also bring lse and delta of 32 queries
  constexpr int kOpBytes = kRows * D * 2;
  constexpr int kSmallOff = 4 * kOpBytes;
  constexpr int kStageBytes = kSmallOff + NSMALL * 256;
  constexpr int LPT = 4;                             // loads of a wavefront per tile
  static_assert(kOpBytes == kKeyWaves * 1024 && kKeyQ % kRows == 0, "one 1 KB load per wavefront and operand");
  static_assert(kKeyLds<D> == kStages * kStageBytes, "");

  const Layer& L = p.L;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

  // Persistent: one item of the work list per iteration.  (Claimed while the one before is worked on, a workgroup with a long item
  // keeps another from those that are free: 3000 tokens, 28 heads 183 -> 215 us.)
  const int n_items = p.klist[1];
  for (;;) {
  __syncthreads();                             // LDS of the previous item is no longer read
  if (threadIdx.x == 0) {
    const int k = atomicAdd(&p.klist[0], 1);
    sItem = k < n_items ? reinterpret_cast<const int4*>(p.klist + kKeyListHeader)[k] : make_int4(-1, 0, 0, 0);
  }
  __syncthreads();
  const int item = __builtin_amdgcn_readfirstlane(sItem.x);
  if (item < 0) break;
  const int bh = item >> 16, ktile = (item >> 3) & 0x1fff, sp = item & 7;
  const int b = bh / L.Hq;
  const int q_begin = __builtin_amdgcn_readfirstlane(sItem.y), n_q = __builtin_amdgcn_readfirstlane(sItem.z);
  const int q_full_pos = __builtin_amdgcn_readfirstlane(sItem.w);   // tiles starting at or after this position need no mask
  const int slot = ktile * kKeyTile + wave * 32 + ln;       // this lane's key slot (< npad by construction)
  int my_first = p.kfirst[(long long)bh * p.npad + slot];

  // resident K and V fragments: B operands, lane = key column
  long long kv_row = (long long)bh * p.npad + slot;
  if constexpr (TILEMAP) {           // the slot's row inside its KV head's token-ordered copy (slots past the map: masked)
    const int t = slot / kTileN;
    const int src = t < p.tile_stride ? p.tile_map[(long long)bh * p.tile_stride + t] : 0;
    kv_row = (long long)(b * L.Hkv + (bh % L.Hq) / L.G) * p.npad_kv + (long long)src * kTileN + slot % kTileN;
  }
  const long long kv_at = (kv_row & ~31ll) * D + lane * 8;
  const T* krow = static_cast<const T*>(p.Kn) + kv_at;
  const T* vrow = static_cast<const T*>(p.Vn) + kv_at;
  bf16x8 kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    kf[ks] = *reinterpret_cast<const bf16x8*>(krow + ks * 512);
    vf[ks] = *reinterpret_cast<const bf16x8*>(vrow + ks * 512);
  }
  // finish every ordinary load here: a compiler-placed wait inside the tile loop would drain the ring
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    asm volatile("" : "+v"(kf[ks]));
    asm volatile("" : "+v"(vf[ks]));
  }
  if (h == 0) sFirst[wave * 32 + ln] = my_first;           // of this wavefront only: read in the masked tiles

  f32x16 dk[NB], dv[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[db][r] = 0.f, dv[db][r] = 0.f;


  const long long q_row = (long long)bh * p.nqpad + (long long)q_begin * kKeyQ;    // first row of this workgroup's tiles
  const T* qn = static_cast<const T*>(p.Qn) + q_row * D;
  const T* gn = static_cast<const T*>(p.dOn) + q_row * D;
  const T* qt = static_cast<const T*>(p.Qt) + q_row * D;
  const T* gt = static_cast<const T*>(p.dOt) + q_row * D;
  const float* small = p.lse2c + q_row + wave % NSMALL * 32;       // every wavefront brings one: the same count of loads for all
  const unsigned delta_off = (unsigned)((p.deltac - p.lse2c) * 4);     // delta lies behind lse (carve_bwd)

  const int n = n_q * (kKeyQ / kRows);
  // u = tile index relative to the workgroup's first (ring position); past the end the last tile comes again, into a stage
  // that nobody reads any more, so that the loads in flight are the same number in every step
  auto issue_part = [&](int u, int op) {
    const unsigned dst = lds_base + (unsigned)(u % kStages) * kStageBytes + op * kOpBytes + wave * 1024;
    const long long tile_off = (long long)min(u, n - 1) * kRows * D;
    gload_lds16((op == 0 ? qn : op == 1 ? gn : op == 2 ? gt : qt) + tile_off + wave * 512, (unsigned)loop_lane() * 16, dst);
  };
  auto issue_small = [&](int u) {
    const unsigned l = (unsigned)loop_lane();
    gload_lds4(small + min(u, n - 1) * kRows, (l < 32 ? l : l - 32) * 4 + (l < 32 ? 0u : delta_off),
               lds_base + (unsigned)(u % kStages) * kStageBytes + kSmallOff + wave % NSMALL * 256);
  };
  auto issue_tile = [&](int u) {
#pragma unroll
    for (int op = 0; op < 4; ++op) issue_part(u, op);
    issue_small(u);
  };

  constexpr int NC = 2 * NB;                   // matrix instructions of a 32-query block in each of the two updates
  constexpr int kAhead = 2;                    // fragment reads run this many of them ahead
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  auto compute_tile = [&](int u, auto with_mask) {
    const int l = loop_lane();
    const unsigned char* stage = smem + (u % kStages) * kStageBytes;
    const unsigned char* st = stage + l * 16;                        // fragments: 16 bytes a lane, in lane order
    int rel = 0;                                     // query positions below rel do not see this lane's key
    if (decltype(with_mask)::value) rel = sFirst[wave * 32 + (l & 31)] - (l >> 5) * 4 - q_begin * kKeyQ - u * kRows;
#pragma unroll
    for (int qb = 0; qb < kRows / 32; ++qb) {
      // S^T and dP^T of the block's 32 queries: chunk c = operand (0: Q, 1: dO), k step
      auto afrag = [&](int c) {
        return *reinterpret_cast<const bf16x8*>(st + (c / KS) * kOpBytes + (qb * KS + c % KS) * 1024);
      };
      // dO, then Q, k-packed: chunk c = operand, 16-query step, 32-column block
      auto cfrag = [&](int c) {
        return *reinterpret_cast<const bf16x8*>(st + (2 + c / NC) * kOpBytes + (qb * NC + c % NC) * 1024);
      };
      const unsigned char* small_b = stage + (l >> 5) * 16 + kSmallOff + qb * 256;
      f32x16 s, dp;
      bf16x8 fa[kAhead];
      bf16x8 pf[2], df[2];
      // weights of four queries: accumulator rows are queries 8 (r/4) + 4 h + r%4 of the block, the column is this
      // lane's key.  Only the query tiles at the causal diagonal of the key tile pay for the position compares.
      // lse of the next four, then delta, is read while these are formed.
      f32x4 next = *reinterpret_cast<const f32x4*>(small_b);
      auto weights = [&](int q4) {
        const f32x4 l4 = next;
        next = *reinterpret_cast<const f32x4*>(small_b + (q4 < 3 ? 32 * (q4 + 1) : 128));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = q4 * 4 + e;
          float pv = fast_exp2(fmaf(s[r], c2, -l4[e]));
          if (decltype(with_mask)::value && qb * 32 + 8 * q4 + e < rel) pv = 0.f;
          s[r] = pv;
        }
      };
      auto ds = [&](int q4) {
        const f32x4 d4 = next;
        if (q4 < 3) next = *reinterpret_cast<const f32x4*>(small_b + 128 + 32 * (q4 + 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) dp[q4 * 4 + e] = s[q4 * 4 + e] * (dp[q4 * 4 + e] - d4[e]);
      };
      constexpr int kPerW = KS / 4, kPerD = NC / 4;      // matrix instructions per quad of weights, of dS
#pragma unroll
      for (int c = 0; c < kAhead; ++c) fa[c] = afrag(c);
#pragma unroll
      for (int c = 0; c < 2 * KS; ++c) {
        __builtin_amdgcn_sched_barrier(0);
        if (c < KS) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c % kAhead], kf[c % KS], c == 0 ? zero16 : s, 0, 0, 0);
        else dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c % kAhead], vf[c % KS], c == KS ? zero16 : dp, 0, 0, 0);
        if (c + kAhead < 2 * KS) fa[c % kAhead] = afrag(c + kAhead);
        else fa[c % kAhead] = cfrag(c + kAhead - 2 * KS);
        if (c >= KS && (c - KS) % kPerW == kPerW - 1) weights((c - KS) / kPerW);      // under the products of dP
        if (qb == 0 && c < 4) issue_part(u + kAheadTiles, c);
      }
      pf[0] = pack8(s, 0);
      pf[1] = pack8(s, 8);
#pragma unroll
      for (int c = 0; c < 2 * NC; ++c) {
        const int db = c % NB;
        __builtin_amdgcn_sched_barrier(0);
        if (c == NC) {
          df[0] = pack8(dp, 0);
          df[1] = pack8(dp, 8);
        }
        if (c < NC) dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c % kAhead], pf[c % NC / NB], dv[db], 0, 0, 0);
        else dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c % kAhead], df[c % NC / NB], dk[db], 0, 0, 0);
        if (c + kAhead < 2 * NC) fa[c % kAhead] = cfrag(c + kAhead);
        if (c < NC && c % kPerD == kPerD - 1) ds(c / kPerD);                          // under the products of dV
        if (qb == 0 && c == 0) issue_small(u + kAheadTiles);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Ring of kStages buffers, one barrier per tile: at the top of step u the tiles up to u + kStages - 2 have
  // been issued; after its barrier everyone is done with tile u-1, whose buffer takes tile u + kStages - 1.
  if (n > 0) {
    wait_vmcnt<0>();
#pragma unroll
    for (int a = 0; a < kAheadTiles; ++a) issue_tile(a);
    const int n_masked = __builtin_amdgcn_readfirstlane(cdiv(min(n * kRows, max(0, q_full_pos - q_begin * kKeyQ)), kRows));
    auto tiles = [&](int from, int to, auto with_mask) {
      for (int u = from; u < to; ++u) {
        wait_vmcnt<(kAheadTiles - 1) * (LPT + 1)>();
        __syncthreads();
        compute_tile(u, with_mask);
      }
    };
    tiles(0, n_masked, std::true_type{});
    tiles(n_masked, n, std::false_type{});
    wait_vmcnt<0>();                           // nothing may land in LDS any more
  }

  // ---- write dK' (scaled) and dV' for this lane's key slot; accumulator rows are d
  const long long out = sp * p.plane + ((long long)bh * p.npad + slot) * D;
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const int d = db * 32 + 8 * q4 + 4 * h;
      const f32x4 x = {dk[db][q4 * 4], dk[db][q4 * 4 + 1], dk[db][q4 * 4 + 2], dk[db][q4 * 4 + 3]};
      const f32x4 y = {dv[db][q4 * 4], dv[db][q4 * 4 + 1], dv[db][q4 * 4 + 2], dv[db][q4 * 4 + 3]};
      *reinterpret_cast<f32x4*>(p.dKp + out + d) = x * L.scale;
      *reinterpret_cast<f32x4*>(p.dVp + out + d) = y;
    }
  }   // items
}

// Key items, then dQ items: a workgroup that finds no key item left goes on with the other list, so that a launch has one tail
// instead of two, filled with the shortest dQ items.  Forward and backward in us, as two launches / one: 28 heads, d = 128, 6000
// tokens 495 / 426 (a budget per head: 398 / 310), 12000 (a budget per head) 887 / 730, 8 heads, 8000 406 / 315, d = 64, 20000
// 1521 / 1479, 32768 6473 / 6460; blocks at d = 64, 8192 663 / 604.  Beside the key items of many heads 256-row dQ items leave no
// CUs idle on short sequences either (two launches, with 32-row dQ items / one): two clips of 3101, d = 64, 165 / 145, 28 heads, d =
// 128, 500 tokens 88 / 79, 1072 107 / 87, 3000 212 / 179, d = 64, 2000 98 / 98.
template <int D, bool TILEMAP, bool FEW_ROWS>
__global__ __launch_bounds__(kKeyThreads, 2) void attn_bwd_bf16_kernel(BwdParams p) {
  static_assert(kKeyThreads == kDqThreads, "one workgroup does both");
  constexpr int kDq = FEW_ROWS ? kDqRowsLds<D> : kDqLds<D>;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kDq > kKeyLds<D> ? kDq : kKeyLds<D>];
  __shared__ int4 sItem;
  __shared__ int sFirst[kKeyTile];
  __shared__ int sTileMap[TILEMAP && !FEW_ROWS ? kBwdMaxMapTiles : 1];
  key_items<D, TILEMAP>(p, smem, sItem, sFirst);
  if constexpr (FEW_ROWS) dq_row_items<D, TILEMAP>(p, smem, sItem);
  else dq_items<D, TILEMAP>(p, smem, sItem, sTileMap);
}

// ------------------------------------------------------------------ dK, dV = sum over the heads of a KV group

// grid: (ceil(N / rows_per_block), B*Hkv); one token row per D/4 lanes.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void attn_bwd_reduce_kernel(BwdParams p, const int* __restrict__ inv,
                                                                  T* __restrict__ dK, T* __restrict__ dV) {
  constexpr int LPR = D / 4;
  constexpr int RPB = kThreads / LPR;
  const Layer& L = p.L;
  const int bg = blockIdx.y, b = bg / L.Hkv, g = bg % L.Hkv;
  const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR;
  const int n = blockIdx.x * RPB + r0;
  if (n >= L.N) return;
  f32x4 ak = {0.f, 0.f, 0.f, 0.f}, av = {0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < L.G; ++j) {
    const int bh = b * L.Hq + g * L.G + j;
    // Slot of token n in the head's list, if it has one: of the other tokens nobody has written the entry, so what it says is
    // looked up in the list (a fill of the map would stand between it and the pass that writes it).
    const int pos = inv[(long long)bh * L.N + n], nkeys = min(p.budget[budget_slot(L.bph, b, bh)], p.b_cap);
    if (pos >= 0 && pos < nkeys && p.list[(long long)bh * p.list_stride + pos] == n) {
      int n_sp = 1;
      if (p.nsplit > 1) {                  // as the key kernel counted: the query tiles from the tile's first visible pair on
        const int first = p.kfirst[(long long)bh * p.npad + pos / kKeyTile * kKeyTile];
        n_sp = key_tile_splits(cdiv(p.q_cnt[bh], kKeyQ) - first / kKeyQ, p.nsplit, p.klist ? p.klist[2] : p.split_len);
      }
      const long long o = ((long long)bh * p.npad + pos) * D + c * 4;
      for (int sp = 0; sp < n_sp; ++sp) {
        ak += *reinterpret_cast<const f32x4*>(p.dKp + sp * p.plane + o);
        av += *reinterpret_cast<const f32x4*>(p.dVp + sp * p.plane + o);
      }
    }
  }
  const long long o = b * L.ks[0] + g * L.ks[1] + (long long)n * L.ks[2] + c * 4;
  if constexpr (sizeof(T) == 2) {
    uint2 wk, wv;
    wk.x = pack_bf16x2(ak[0], ak[1]);
    wk.y = pack_bf16x2(ak[2], ak[3]);
    wv.x = pack_bf16x2(av[0], av[1]);
    wv.y = pack_bf16x2(av[2], av[3]);
    *reinterpret_cast<uint2*>(dK + o) = wk;
    *reinterpret_cast<uint2*>(dV + o) = wv;
  } else {
    *reinterpret_cast<f32x4*>(dK + o) = ak;
    *reinterpret_cast<f32x4*>(dV + o) = av;
  }
}

struct BwdWs {
  void *Kn, *Vn, *Kt, *Qt, *dOt, *Qn, *dOn;
  int* kidx;
  float *lse2c, *deltac, *dKp, *dVp;
  int* sched;
  int *qvis, *kfirst, *inv, *klist;
  int *vbudget, *tile_map;                // in-place block lists only, as kidx
};

// Block lists walked in place (omni_block_attn_bwd): ascending block ids per head, one budget per batch item.
struct BlockLists {
  const int* blk_idx;
  const int* blk_budget;
  int blk_cap, block;
};

// Which dQ items, by the shape only (the gathered and the in-place lists of a layer take the same ones).  Backward call in us,
// 256-row items / 32-row ones; a third of the queries and half of the keys kept, or all (full).  d = 128: 1 head 8192 156 / 123,
// 24000 453 / 351 and (full) 8192 259 / 129, 24000 848 / 604; 2 heads (full) 12000 429 / 336; 4 heads 6000 134 / 109 and (full)
// 230 / 200; 8 heads 3100 88 / 80 and (full) 144 / 148; above the line 8 heads 4096 110 / 92 but (full) 186 / 223, 4 heads 12000
// 252 / 214 but (full) 526 / 766, 14 heads 2048 76 / 73 but (full) 135 / 150, 28 heads 1072 65 / 65 and (full) 108 / 121.  d = 64: 1
// head 32768 410 / 328 and (full) 725 / 582, 4 heads 8192 120 / 88 and (full) 207 / 178, 8 heads 4096 80 / 62 and (full) 122 /
// 118; above the line 4 heads 12000 165 / 120 but (full) 321 / 361, 8 heads 6000 102 / 86 but (full) 182 / 223, 14 heads 3100 76 /
// 73 but (full) 122 / 142.
inline bool bwd_few_rows(const Layer& L) {
  const long long heads = (long long)L.B * L.Hq;
  return heads <= 8 && heads * L.N <= (L.D == 128 ? 26000 : 40000);
}

constexpr int kKeyHeadGroup = 7;
int g_key_split_len = kKeySplitLen;          // omni_debug_key_split_len: tests split short key tiles too
// slots of the key kernel's dispatch order
size_t key_list_slots(const Layer& L, int npad) {
  return (size_t)cdiv(L.B * L.Hq, kKeyHeadGroup) * kKeyHeadGroup * (npad / kKeyTile);
}

// npad_kv > 0: Kn, Vn, Kt hold every KV head once ([B*Hkv, npad_kv, D], the in-place block lists) instead of one
// gathered copy per query head; cap_tiles = key tiles of a head's list then.
BwdWs carve_bwd(Arena& a, const Layer& L, int dtype, int npad, int nqpad, int npad_kv = 0, int cap_tiles = 0) {
  BwdWs w;
  const size_t es = dtype == OMNI_BF16 ? 2 : 4;
  const size_t BH = (size_t)L.B * L.Hq;
  const size_t krows = BH * npad, qrows = BH * nqpad;
  const size_t kvrows = npad_kv > 0 ? (size_t)L.B * L.Hkv * npad_kv : krows;
  w.Kn = a.take<unsigned char>(kvrows * L.D * es);
  w.Vn = a.take<unsigned char>(kvrows * L.D * es);
  const bool copies = dtype == OMNI_BF16 || f32_short(L);
  const size_t planes = copies ? kKeyMaxSplits : 1;
  w.Kt = a.take<unsigned char>(copies ? kvrows * L.D * es : 4);
  w.Qt = a.take<unsigned char>(copies ? qrows * L.D * es : 4);
  w.dOt = a.take<unsigned char>(copies ? qrows * L.D * es : 4);
  w.Qn = a.take<unsigned char>(copies ? qrows * L.D * es : 4);
  w.dOn = a.take<unsigned char>(copies ? qrows * L.D * es : 4);
  w.kidx = a.take<int>(npad_kv > 0 ? krows : 4);
  w.lse2c = a.take<float>(qrows);
  w.deltac = a.take<float>(qrows);
  w.dKp = a.take<float>(planes * krows * L.D);
  w.dVp = a.take<float>(planes * krows * L.D);
  w.sched = a.take<int>(sched_ints(L.B * L.Hq, L.N, dtype == OMNI_BF16 ? kDqTileM : kTileM));
  w.qvis = a.take<int>(BH * L.N);
  w.kfirst = a.take<int>(krows);
  w.inv = a.take<int>(BH * L.N);
  // a tile's splits are no more than its query tiles
  w.klist = a.take<int>(kKeyListHeader + key_list_slots(L, npad) * std::min(kKeyMaxSplits, cdiv(L.N, kKeyQ)) * kKeyItemInts);
  w.vbudget = a.take<int>(L.B);
  w.tile_map = a.take<int>(npad_kv > 0 ? BH * cap_tiles : 4);
  return w;
}

// Rows of a head's packed buffers: whole workgroup tiles, and never a multiple of 4096 rows -- with a
// power-of-two stride between the heads, workgroups that stream different heads at the same tile index hit the
// same cache sets and memory channels.
int bwd_npad(int b_cap) {                     // a multiple of kKeyTile
  int n = (int)align_up(b_cap, kKeyTile);
  if (n % 4096 == 0) n += kKeyTile;
  return n;
}
int bwd_nqpad(const Layer& L) {
  int n = (int)align_up(L.N, kTileM);
  if (n % 4096 == 0) n += kTileM;
  return n;
}

int bwd_npad_kv(const Layer& L) { return (int)align_up(L.N, kTileN); }

// BLOCKS (bf16 only): kv_idx / budget / b_cap are ignored and the key lists are the block lists `blk`, walked in place.
template <typename T, int D, bool BLOCKS>
int launch_bwd(const Layer& L, const void* Q, const void* K, const void* V, const void* O, const void* dO,
               const float* lse, const int* q_idx, const int* q_cnt, const int* kv_idx, const int* budget, int b_cap,
               void* dQ, void* dK, void* dV, void* ws, hipStream_t st, const BlockLists* blk = nullptr) {
  constexpr int dt = sizeof(T) == 2 ? OMNI_BF16 : OMNI_F32;
  static_assert(!BLOCKS || sizeof(T) == 2, "block lists run in bf16");
  Arena a(ws);
  const int cap_keys = BLOCKS ? blk->blk_cap * blk->block : b_cap;
  const int npad = bwd_npad(cap_keys), nqpad = bwd_nqpad(L);
  const int npad_kv = BLOCKS ? bwd_npad_kv(L) : 0;
  BwdWs w = carve_bwd(a, L, dt, npad, nqpad, npad_kv, cap_keys / kTileN);
  constexpr bool kFast = sizeof(T) == 2;
  constexpr int tile_m = kFast ? kDqTileM : kTileM;
  const bool split = !kFast && f32_short(L);           // fp32 on short sequences: no work list
  const bool copies = kFast || split;                  // fp32 on long sequences: only K and V, row by row
  const bool few_rows = kFast && short_route(bwd_few_rows(L));       // dQ items of 32 rows: no work list either
  int rc = check_work_list(L, tile_m);
  if (rc != OMNI_OK) return rc;
  // the bf16 key kernel's list: heads and key tiles in 16 and 13 bits of an item
  if (kFast && (L.B * L.Hq >= 32768 || npad / kKeyTile >= 8192))
    OMNI_FAIL(OMNI_ERR_UNSUPPORTED, "key work list: too many heads or key tiles");
  PackKv kv{};
  kv.K = K;
  kv.V = V;
  kv.Kn = w.Kn;
  kv.Vn = w.Vn;
  kv.Kt = copies ? w.Kt : nullptr;
  kv.k_frag = split;
  if constexpr (BLOCKS) {
    // K, V (fragment order) and K (k-packed) of every KV head once, in token order: shared by the heads of a group
    kv.b_cap = L.N;
    kv.npad = npad_kv;
    kv.pad_to = kTileN;
    // token lists of the selected blocks (causal bounds, the reduction's slot map), rows npad apart, and the tile map
    rc = run_expand_blocks(L, blk->blk_idx, blk->blk_budget, blk->blk_cap, blk->block, w.kidx, w.vbudget, npad, st, w.tile_map,
                           npad_kv / kTileN - 1);
    if (rc != OMNI_OK) return rc;
    kv_idx = w.kidx;
    budget = w.vbudget;
    b_cap = npad;                             // the lists' row pitch; their lengths are in vbudget
  } else {
    kv.per_q_head = 1;
    kv.src_idx = kv_idx;
    kv.idx_stride = b_cap;
    kv.budget = budget;
    kv.b_cap = b_cap;
    kv.npad = npad;
    kv.pad_to = kKeyTile;
  }
  PackQ pq{};
  pq.Q = Q;
  pq.O = O;
  pq.dO = dO;
  pq.lse = lse;
  pq.q_idx = q_idx;
  pq.q_cnt = q_cnt;
  pq.nqpad = nqpad;
  if (copies) {
    pq.Qt = w.Qt;
    pq.dOt = w.dOt;
    pq.Qn = w.Qn;
    pq.dOn = w.dOn;
  }
  pq.lse2c = w.lse2c;
  pq.deltac = w.deltac;
  BwdParams p;
  p.Q = Q;
  p.dO = dO;
  p.L = L;
  p.q_idx = q_idx;
  p.q_cnt = q_cnt;
  p.budget = budget;
  p.b_cap = b_cap;
  p.npad = npad;
  p.nqpad = nqpad;
  p.Kn = w.Kn;
  p.Vn = w.Vn;
  p.Kt = w.Kt;
  p.Qt = w.Qt;
  p.dOt = w.dOt;
  p.Qn = w.Qn;
  p.dOn = w.dOn;
  p.lse2c = w.lse2c;
  p.deltac = w.deltac;
  p.dKp = w.dKp;
  p.dVp = w.dVp;
  p.nsplit = kFast || split ? kKeyMaxSplits : 1;
  p.split_len = sizeof(T) == 2 ? g_key_split_len : kKeySplitLenF32;
  p.plane = (long long)L.B * L.Hq * npad * D;
  p.dQ = dQ;
  p.klist = nullptr;
  p.list = kv_idx;
  p.list_stride = b_cap;
  p.sched = w.sched;
  p.qvis = w.qvis;
  p.kfirst = w.kfirst;
  p.tile_map = w.tile_map;
  p.tile_stride = cap_keys / kTileN;
  p.npad_kv = BLOCKS ? npad_kv : npad;
  Bounds bn{};                                 // masks by position, slot map, cleared rows, the dQ work items
  bn.q_idx = q_idx;
  bn.q_cnt = q_cnt;
  bn.klist = kv_idx;
  bn.klist_stride = b_cap;
  bn.budget = budget;
  bn.b_cap = b_cap;
  bn.npad = npad;
  bn.qvis = w.qvis;
  bn.kfirst = w.kfirst;
  bn.inv = w.inv;
  bn.X = dQ;
  bn.elem_bytes = sizeof(T);
  bn.tile_m = tile_m;
  bn.sched = split || few_rows ? nullptr : w.sched;
  p.order_off = sched_order_off(L.B * L.Hq, L.N, tile_m);
  if (split) {                                 // no list at all: one launch
    rc = run_prepare(L, dt, true, &kv, &pq, &bn, nullptr, nullptr, st);
  } else {                                     // the lists, a few serial workgroups, hide under the packs
    // Dispatch order of the key items: heads in groups of 7, key tile by key tile inside a group.  Head after head leaves the
    // long first key tiles of the last heads for the end, all heads at once spreads 28 query streams over the caches, and group
    // sizes that share a factor with the 8 XCDs (workgroup i runs on XCD i mod 8) pin heads to XCDs and unbalance them.  At 32k, when
    // dK' and dV' were kernels of their own (the two together): 3.9 ms, 4.4 ms, groups of 8 5.6 ms, groups of 7 3.4 ms.
    KeyList kl{};
    kl.q_cnt = q_cnt;
    kl.budget = budget;
    kl.b_cap = b_cap;
    kl.npad = npad;
    kl.kfirst = w.kfirst;
    kl.head_group = kKeyHeadGroup;
    kl.nsplit = p.nsplit;
    kl.split_len = p.split_len;
    kl.key_wgs = persistent_grid() / 2;        // one workgroup per CU (its LDS ring fills it)
    kl.n_slots = (int)key_list_slots(L, npad);
    kl.klist = w.klist;
    if (kFast) p.klist = w.klist;
    const Order order = make_order(L, q_cnt, tile_m, w.sched);
    rc = run_prepare(L, dt, true, nullptr, nullptr, &bn, nullptr, nullptr, st);
    if (rc != OMNI_OK) return rc;
    rc = run_prepare(L, dt, true, &kv, &pq, nullptr, few_rows ? nullptr : &order, kFast ? &kl : nullptr, st);
  }
  if (rc != OMNI_OK) return rc;
  {
    ProfScope prof__(kProfBwdDkDv, st);
    if constexpr (sizeof(T) == 2) {
      const dim3 grid((unsigned)persistent_grid() / 2);
      if (few_rows) hipLaunchKernelGGL((attn_bwd_bf16_kernel<D, BLOCKS, true>), grid, dim3(kKeyThreads), 0, st, p);
      else hipLaunchKernelGGL((attn_bwd_bf16_kernel<D, BLOCKS, false>), grid, dim3(kKeyThreads), 0, st, p);
    } else {
      const unsigned heads = (unsigned)(L.B * L.Hq), key_blocks = heads * (unsigned)(npad / 32) * kKeyMaxSplits;
      if (split)
        hipLaunchKernelGGL((attn_bwd_f32_kernel<D>), dim3(key_blocks + heads * (unsigned)cdiv(L.N, 32)), dim3(kF32Threads<D>), 0, st,
                           p, (int)key_blocks);
      else
        hipLaunchKernelGGL((attn_bwd_key_f32_long_kernel<D>), dim3(npad / kF32Keys, L.B * L.Hq), dim3(kThreads), 0, st, p);
    }
    OMNI_LAUNCH_CHECK();
  }
  if constexpr (!kFast) {
    if (!split) {
      ProfScope prof__(kProfBwdDq, st);
      hipLaunchKernelGGL((attn_bwd_dq_f32_long_kernel<D>), dim3(persistent_grid() / 2), dim3(kThreads), 0, st, p);
      OMNI_LAUNCH_CHECK();
    }
  }
  {
    ProfScope prof__(kProfBwdReduce, st);
    constexpr int RPB = kThreads / (D / 4);
    hipLaunchKernelGGL((attn_bwd_reduce_kernel<T, D>), dim3(cdiv(L.N, RPB), L.B * L.Hkv), dim3(kThreads), 0, st, p,
                       w.inv, static_cast<T*>(dK), static_cast<T*>(dV));
    OMNI_LAUNCH_CHECK();
  }
  return OMNI_OK;
}

}  // namespace

void set_key_split_len(int tiles) { g_key_split_len = tiles > 0 ? tiles : kKeySplitLen; }

size_t attn_bwd_ws(const Layer& L, int dtype, int b_cap) {
  Arena a(nullptr);
  carve_bwd(a, L, dtype, bwd_npad(b_cap), bwd_nqpad(L));
  return a.used();
}

int run_attn_bwd(const Layer& L, int dtype, const void* Q, const void* K, const void* V, const void* O,
                 const void* dO, const float* lse, const int* q_idx, const int* q_cnt, const int* kv_idx,
                 const int* budget, int b_cap, void* dQ, void* dK, void* dV, void* ws, hipStream_t st) {
  if (dtype == OMNI_BF16) {
    if (L.D == 128)
      return launch_bwd<u16, 128, false>(L, Q, K, V, O, dO, lse, q_idx, q_cnt, kv_idx, budget, b_cap, dQ, dK, dV, ws, st);
    return launch_bwd<u16, 64, false>(L, Q, K, V, O, dO, lse, q_idx, q_cnt, kv_idx, budget, b_cap, dQ, dK, dV, ws, st);
  }
  if (L.D == 128)
    return launch_bwd<float, 128, false>(L, Q, K, V, O, dO, lse, q_idx, q_cnt, kv_idx, budget, b_cap, dQ, dK, dV, ws, st);
  return launch_bwd<float, 64, false>(L, Q, K, V, O, dO, lse, q_idx, q_cnt, kv_idx, budget, b_cap, dQ, dK, dV, ws, st);
}

int attn_bwd_blocks_max_keys() { return kBwdMaxMapTiles * kTileN; }

size_t attn_bwd_blocks_ws(const Layer& L, int cap_keys) {
  Arena a(nullptr);
  carve_bwd(a, L, OMNI_BF16, bwd_npad(cap_keys), bwd_nqpad(L), bwd_npad_kv(L), cap_keys / kTileN);
  return a.used();
}

int run_attn_bwd_blocks(const Layer& L, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const float* lse, const int* q_idx, const int* q_cnt, const int* blk_idx, const int* blk_budget,
                        int blk_cap, int block, void* dQ, void* dK, void* dV, void* ws, hipStream_t st) {
  const BlockLists blk{blk_idx, blk_budget, blk_cap, block};
  if (L.D == 128)
    return launch_bwd<u16, 128, true>(L, Q, K, V, O, dO, lse, q_idx, q_cnt, nullptr, nullptr, 0, dQ, dK, dV, ws, st, &blk);
  return launch_bwd<u16, 64, true>(L, Q, K, V, O, dO, lse, q_idx, q_cnt, nullptr, nullptr, 0, dQ, dK, dV, ws, st, &blk);
}

}  // namespace omni
