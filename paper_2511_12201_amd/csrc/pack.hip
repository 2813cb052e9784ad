// Gather / re-layout passes that feed the attention kernels (HBM-bound copies).
//
// pack_kv: per head, the selected K/V rows are gathered into dense buffers and
// padded with zero rows to whole 64-key tiles (who sees a slot is read from the
// key lists themselves: bounds_block, sched_dev.h).  Layouts: "fragment order"
// [32-row block][k step][lane] of 16 bytes, lane = 32 h + row (a k step is 16 elements of
// bf16, 8 of fp32): the A or B operand of a 32x32 MFMA that contracts over d, a kilobyte
// per operand with the lanes side by side, in memory and in LDS alike (no swizzle, one
// address register for all of a tile's fragments); and "k-packed" [16-slot group][d / 32][half h][d % 32][8 slots]
// with slot(group,h,j) = 16 group + 8 (j/4) + 4 h + j%4 -- the order in which a
// 32x32 MFMA accumulator holds its rows -- so that the operand of a GEMM that
// contracts over the slots is one 16-byte read per lane.  The k-packed
// V (the forward's operand; the backward does not use it) is written in f16: the
// forward multiplies its f16-rounded weights with it.  fp32 inputs on long sequences
// (k_frag false): rows as they are.  fp32 inputs, k-packed: [32-slot block][q4][d / 32][h][d % 32][4
// slots], slot = 8 q4 + 4 h + e: the fp32 MFMA takes one element per lane, four of them
// arrive with one 16-byte read.
//
// pack_q: for the backward pass, the kept rows of Q and dO in the k-packed
// layout (contraction over queries) and in fragment order, plus per kept row
// lse * log2(e) and delta = rowsum(dO * O).
//
// Both, and the passes over the lists (sched_dev.h), are roles of one kernel: on short sequences a launch that does nothing
// takes 4 us, as long as most of these passes, and on long ones the serial work-list blocks hide under the packs.  Launches
// one by one -> as roles and the whole call in us, when that was done: one-call prefill of 1072 tokens 12 -> 11, 87.5 -> 84.4; fp32 forward and backward,
// 1024 tokens, 9 -> 6, 87 -> 75; two clips of 3101 at d = 64, 10 -> 7, 178 -> 168; forward of 16391 tokens 4 -> 3, 430 ->
// 427; blocks at 16k, forward and backward, 24 -> 18, 3044 -> 3001.
#include "common.h"
#include "kernels.h"
#include "sched_dev.h"

#include <algorithm>

namespace omni {

namespace {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

// Eight bf16 values as f16.  Every bf16 value of magnitude in [2^-14, 65504] is an f16 value (8 significant bits
// into 11); smaller ones land on the f16 subnormal grid (absolute error below 3e-8), larger ones saturate at 65504
// (the conversion rounds towards zero, which never produces an infinity from a finite value).
__device__ __forceinline__ u32x4 bf16x8_to_f16x8(const u32x4& x) {
  u32x4 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float lo = __uint_as_float(x[j] << 16), hi = __uint_as_float(x[j] & 0xffff0000u);
    const auto pk = __builtin_amdgcn_cvt_pkrtz(lo, hi);
    r[j] = __builtin_bit_cast(unsigned, pk);
  }
  return r;
}

// Unit t of a 64-slot tile in the bf16 k-packed order: (16-slot group, half, 8-wide d chunk), 128 bytes of output, the units in
// the order of the output.
template <int D>
__device__ __forceinline__ void packed_unit(int t, int& grp, int& h, int& dc) {
  constexpr int NB = D / 32;
  dc = (t >> 3) % NB * 4 + (t & 3);
  h = (t >> 2) & 1;
  grp = t / (8 * NB);
}

// 8 rows x 8 bf16 (one 16-byte chunk per row) of every lane -> its 8 columns x 8 rows, 128 bytes; the wavefront's 8 KB are
// contiguous in lane order and leave through `lds` (8 KB of its own) as eight whole kilobytes: straight from the registers a
// store would touch 64 cache lines with 16 bytes each.
__device__ __forceinline__ void transpose8x8_store(const u32x4 (&in)[8], u16* wave_dst, unsigned char* lds) {
  const int l = lane_id();
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    unsigned w[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const unsigned a = in[2 * jj][e >> 1], b = in[2 * jj + 1][e >> 1];
      w[jj] = __builtin_amdgcn_perm(b, a, (e & 1) ? 0x07060302u : 0x05040100u);       // high or low halves of a, then b
    }
    *reinterpret_cast<u32x4*>(lds + (l * 8 + (e ^ (l & 7))) * 16) = u32x4{w[0], w[1], w[2], w[3]};
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int p = j * 64 + l, from = p >> 3;
    *reinterpret_cast<u32x4*>(wave_dst + p * 8) = *reinterpret_cast<const u32x4*>(lds + (from * 8 + ((p & 7) ^ (from & 7))) * 16);
  }
}

// 4 rows x 4 floats -> 4 columns x 4 rows in the fp32 k-packed order; dst: the 32-slot block, unit = q4 * 2 + h
template <int D>
__device__ __forceinline__ void transpose4x4_store(const u32x4 (&in)[4], float* dst, int q4, int h, int dc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int d = dc * 4 + e;
    const u32x4 o = {in[0][e], in[1][e], in[2][e], in[3][e]};
    *reinterpret_cast<u32x4*>(dst + (((q4 * (D / 32) + d / 32) * 2 + h) * 32 + d % 32) * 4) = o;
  }
}

// grid: (npad/64, BHx).  The lists are read, also where selection and attention are one call: forming a tile's 64 entries
// here from the scores and the head's cut saves the list writer nothing (it still runs, for the queries) and puts a search,
// a scan and a ranking before every gather.  One-call prefill in us, formed here / read: 1072 tokens 93.3 / 90.6, 4096:
// 153 / 148, 16384: 526 / 520, 65536: 4797 / 4792; 8 heads, 16384: 313 / 302.
// bf16: two wavefronts per output, so that a thread has one batch of loads and the outputs do not wait for each other.  (The
// copies by all threads, then the transposes by those that had one, was a second memory latency for every workgroup.)
// Layer in us, before / after, with the same change in pack_q below: forward, 1072 tokens 89.5 / 87.3, 16391: 432.5 / 430.3,
// d = 64, 3000: 41.7 / 40.1; forward and backward, two clips of 3101, d = 64: 202.4 / 198.3, 32768: 7364 / 7339.  (d threads
// per output: 8192 at d = 64 2.5 % slower.)
// Bound on long sequences: the writes (the K/V of the KV heads, read once per query head, come from the caches), so every
// store instruction covers whole lines (transpose8x8_store; 128-byte pieces in the copies).  28 heads, d = 128, stores of 16
// bytes to 64 lines at once / whole lines: for the forward 16391 46.9 / 39.4 us, 32768 91 / 72 us (253 MB written: 3.5
// TB/s), for the backward 109 / 97 us, pack_q there 168 / 131 us.
constexpr int kOutThreads = 128;
template <int WAVES>
struct PackShared {                      // exchange areas of the wavefronts that write k-packed copies (bf16)
  __attribute__((aligned(16))) unsigned char t[WAVES][8192];
  int idx[64];
};
template <>
struct PackShared<0> {
  int idx[64];
};
template <typename T, int D, typename Shared>
__device__ __forceinline__ void pack_kv_block(const Layer& L, const PackKv& p, int tile, int bhx, Shared& sh) {
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int E = Elem<T>::kPer16B;
  constexpr int CPR = D / E;
  const T *K = static_cast<const T*>(p.K), *V = static_cast<const T*>(p.V);
  T *Kn = static_cast<T*>(p.Kn), *Vn = static_cast<T*>(p.Vn), *Kt = static_cast<T*>(p.Kt), *Vt = static_cast<T*>(p.Vt);
  const int npad = p.npad, k_frag = p.k_frag, per_q_head = p.per_q_head;
  int* sIdx = sh.idx;
  const int H = per_q_head ? L.Hq : L.Hkv;
  const int b = bhx / H, hx = bhx % H;
  const int g = per_q_head ? hx / L.G : hx;
  const int nkeys = p.budget ? min(p.budget[per_q_head ? budget_slot(L.bph, b, bhx) : b], p.b_cap) : L.N;
  if (tile * kTileN >= (int)align_up((size_t)max(nkeys, 0), (size_t)p.pad_to)) return;   // consumers read whole pad_to-slot groups
  if (threadIdx.x < kTileN) {
    const int slot = tile * kTileN + threadIdx.x;
    int id = kPadKeyIndex;
    if (slot < nkeys) id = p.src_idx ? p.src_idx[(long long)bhx * p.idx_stride + slot] : slot;
    sIdx[threadIdx.x] = id;
  }
  __syncthreads();
  const T* kbase = K + b * L.ks[0] + g * L.ks[1];
  const T* vbase = V + b * L.ks[0] + g * L.ks[1];
  const long long tile_off = ((long long)bhx * npad + tile * kTileN) * D;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  if constexpr (kBf16) {
    const int t = threadIdx.x % kOutThreads;
    int unit = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kOutThreads));
    // fragment order: a wavefront takes 8 rows of 128 bytes at a time and leaves 8 columns of 128 bytes
    auto copy = [&](const T* src, T* dst) {
      constexpr int kEach = kTileN * CPR / kOutThreads;
      u32x4 in[kEach];
      int at[kEach];
#pragma unroll
      for (int j = 0; j < kEach; ++j) {
        const int u = j * (kOutThreads / 64) + t / 64, row = u % 8 * 8 + (t & 7), chunk = u / 8 * 8 + (t >> 3 & 7);
        const int id = sIdx[row];
        at[j] = (row / 32 * 32 * CPR + chunk * 32 + row % 32) * E;
        in[j] = zero;
        if (id != kPadKeyIndex) in[j] = *reinterpret_cast<const u32x4*>(src + (long long)id * L.ks[2] + chunk * E);
      }
#pragma unroll
      for (int j = 0; j < kEach; ++j) *reinterpret_cast<u32x4*>(dst + tile_off + at[j]) = in[j];
    };
    // a thread transposes 8 slots x 8 of d in registers
    auto transposed = [&](const T* src, T* dst, bool f16) {
      if (t >= D) return;
      u32x4 in[8];
      int grp, h, dc;
      packed_unit<D>(t, grp, h, dc);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int id = sIdx[16 * grp + 8 * (j >> 2) + 4 * h + (j & 3)];
        in[j] = zero;
        if (id != kPadKeyIndex) in[j] = *reinterpret_cast<const u32x4*>(src + (long long)id * L.ks[2] + dc * 8);
      }
      if (f16) {                                       // the forward multiplies its weights and V in f16
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] = bf16x8_to_f16x8(in[j]);
      }
      transpose8x8_store(in, reinterpret_cast<u16*>(dst) + tile_off + t / 64 * 4096, sh.t[t / 64]);
    };
    if (Kn && unit-- == 0) copy(kbase, Kn);
    if (Vn && unit-- == 0) copy(vbase, Vn);
    if (Kt && unit-- == 0) transposed(kbase, Kt, false);
    if (Vt && unit-- == 0) transposed(vbase, Vt, true);
  } else {
#pragma unroll                                      // all loads of a thread in flight together
    for (int c = threadIdx.x; c < kTileN * CPR; c += kThreads) {
      const int row = k_frag ? c / (32 * CPR) * 32 + (c & 31) : c / CPR, chunk = k_frag ? c / 32 % CPR : c % CPR;
      const int id = sIdx[row];
      const long long src = (long long)id * L.ks[2] + chunk * E;
      u32x4 k = zero, v = zero;
      if (Kn && id != kPadKeyIndex) k = *reinterpret_cast<const u32x4*>(kbase + src);
      if (Vn && id != kPadKeyIndex) v = *reinterpret_cast<const u32x4*>(vbase + src);
      if (Kn) *reinterpret_cast<u32x4*>(Kn + tile_off + c * E) = k;
      if (Vn) *reinterpret_cast<u32x4*>(Vn + tile_off + c * E) = v;
    }
    // work item = (tensor, 4-slot group, 4-wide d chunk)
    constexpr int kItems = (kTileN / 4) * (D / 4);
    for (int it0 = threadIdx.x; it0 < 2 * kItems; it0 += kThreads) {
      const int which = it0 / kItems, dc = it0 % (D / 4), grp = it0 % kItems / (D / 4);
      T* dst_t = which ? Vt : Kt;
      if (!dst_t) continue;
      const T* src = which ? vbase : kbase;
      u32x4 in[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int id = sIdx[grp * 4 + j];
        in[j] = zero;
        if (id != kPadKeyIndex) in[j] = *reinterpret_cast<const u32x4*>(src + (long long)id * L.ks[2] + dc * 4);
      }
      transpose4x4_store<D>(in, reinterpret_cast<float*>(dst_t) + tile_off + grp / 8 * 32 * D, grp / 2 % 4, grp & 1, dc);
    }
  }
}

// Tile t covers kept positions [64 t, 64 t + 64).
// bf16: the wavefronts past the first four write the k-packed copies meanwhile, D threads each.
template <typename T, int D, typename Shared>
__device__ __forceinline__ void pack_q_block(const Layer& L, const PackQ& p, int tile, int bh, Shared& sh) {
  const T *Q = static_cast<const T*>(p.Q), *O = static_cast<const T*>(p.O), *dO = static_cast<const T*>(p.dO);
  T *Qt = static_cast<T*>(p.Qt), *dOt = static_cast<T*>(p.dOt), *Qn = static_cast<T*>(p.Qn), *dOn = static_cast<T*>(p.dOn);
  const int nqpad = p.nqpad;
  int* sIdx = sh.idx;
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int E = Elem<T>::kPer16B;
  constexpr int LPR = D / E;
  constexpr int RPP = kThreads / LPR;
  const int b = bh / L.Hq, i = bh % L.Hq;
  const int nq = p.q_cnt[bh];
  if (tile * 64 >= nq) return;
  if (threadIdx.x < 64) {
    const int pos = tile * 64 + threadIdx.x;
    sIdx[threadIdx.x] = pos < nq ? p.q_idx[(long long)bh * L.N + pos] : -1;
  }
  __syncthreads();
  const long long head_off = b * L.qs[0] + i * L.qs[1];
  // delta = rowsum(dO * O), lse in log2 units; rows that contribute nothing get lse = +inf (P = 0)
  const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR;
  if (!kBf16 || threadIdx.x < kThreads) {
#pragma unroll                                      // all loads of a thread in flight together
    for (int rb = 0; rb < 64; rb += RPP) {
      const int r = rb + r0;
      const int row = sIdx[r];
      float dot = 0.f;
      u32x4 g = {0u, 0u, 0u, 0u}, qc = {0u, 0u, 0u, 0u};
      if (row >= 0) {
        const u32x4 a = *reinterpret_cast<const u32x4*>(O + head_off + (long long)row * L.qs[2] + c * E);
        g = *reinterpret_cast<const u32x4*>(dO + head_off + (long long)row * L.qs[2] + c * E);
        if (Qn) qc = *reinterpret_cast<const u32x4*>(Q + head_off + (long long)row * L.qs[2] + c * E);
        float av[E], gv[E];
        unpack16(a, av, (const T*)nullptr);
        unpack16(g, gv, (const T*)nullptr);
#pragma unroll
        for (int e = 0; e < E; ++e) dot = fmaf(av[e], gv[e], dot);
      }
      if (Qn) {                                   // packed copies in fragment order (pad rows zero)
        const long long o = ((long long)bh * nqpad + tile * 64 + r / 32 * 32) * D + (c * 32 + r % 32) * E;
        *reinterpret_cast<u32x4*>(Qn + o) = qc;
        *reinterpret_cast<u32x4*>(dOn + o) = g;
      }
#pragma unroll
      for (int o = LPR / 2; o > 0; o >>= 1) dot += __shfl_xor(dot, o, 64);
      if (c == 0) {
        const long long o = (long long)bh * nqpad + tile * 64 + r;
        float l2 = INFINITY;
        if (row >= 0) {
          const float lv = p.lse[(long long)bh * L.N + row];
          l2 = lv == -INFINITY ? INFINITY : lv * kLog2e;
        }
        p.lse2c[o] = l2;
        p.deltac[o] = row >= 0 ? dot : 0.f;
      }
    }
  }
  if constexpr (kBf16) {
    constexpr int kItems = (64 / 16) * 2 * (D / 8);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const long long tile_off = ((long long)bh * nqpad + tile * 64) * D;
    static_assert(kItems == D, "one item per thread");
    if (threadIdx.x >= kThreads) {
      const int it0 = threadIdx.x - kThreads, which = it0 / kItems, it = it0 % kItems;
      const T* src = (which ? dO : Q) + head_off;
      T* dst_t = which ? dOt : Qt;
      int grp, h, dc;
      packed_unit<D>(it, grp, h, dc);
      u32x4 in[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int row = sIdx[16 * grp + 8 * (j >> 2) + 4 * h + (j & 3)];
        in[j] = zero;
        if (row >= 0) in[j] = *reinterpret_cast<const u32x4*>(src + (long long)row * L.qs[2] + dc * 8);
      }
      transpose8x8_store(in, reinterpret_cast<u16*>(dst_t) + tile_off + it / 64 * 4096, sh.t[it0 / 64]);
    }
  } else {
    constexpr int kItems = (64 / 4) * (D / 4);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const long long tile_off = ((long long)bh * nqpad + tile * 64) * D;
    for (int it0 = threadIdx.x; it0 < 2 * kItems; it0 += kThreads) {
      const int which = it0 / kItems, dc = it0 % (D / 4), grp = it0 % kItems / (D / 4);
      const T* src = (which ? dO : Q) + head_off;
      T* dst_t = which ? dOt : Qt;
      if (!dst_t) break;                               // both or neither
      u32x4 in[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = sIdx[grp * 4 + j];
        in[j] = zero;
        if (row >= 0) in[j] = *reinterpret_cast<const u32x4*>(src + (long long)row * L.qs[2] + dc * 4);
      }
      transpose4x4_store<D>(in, reinterpret_cast<float*>(dst_t) + tile_off + grp / 8 * 32 * D, grp / 2 % 4, grp & 1, dc);
    }
  }
}

// grid: the blocks of the roles one after the other, those that take longest first
struct Roles {
  int order, keys, bounds, q;            // blocks of each; the rest is K/V tiles
  int bounds_x, q_x, kv_x;
};
template <typename T, int D, int NT, bool Q_ROLE>
__global__ __launch_bounds__(NT) void prepare_kernel(Layer L, Roles r, PackKv kv, PackQ q, Bounds bn, Order od, KeyList kl) {
  constexpr int kWaves = sizeof(T) == 4 ? 0 : Q_ROLE ? 2 * D / 64 : D / 64;       // Q and dO at once, or V
  __shared__ union {
    PackShared<kWaves> pack;
    OrderShared<NT> order;
    int wave_cnt[NT / 64];
  } sh;
  int i = blockIdx.x;
  if (i < r.order) return order_block<NT>(od, i, sh.order);
  i -= r.order;
  if (i < r.keys) return key_list_block<NT>(L, kl, sh.wave_cnt);
  i -= r.keys;
  const int BH = L.B * L.Hq;
  if (i < r.bounds) return bounds_block<NT>(L, bn, i % r.bounds_x, i / r.bounds_x % BH, i / r.bounds_x / BH);
  i -= r.bounds;
  if constexpr (Q_ROLE) {
    if (i < r.q) return pack_q_block<T, D>(L, q, i % r.q_x, i / r.q_x, sh.pack);
    i -= r.q;
  }
  pack_kv_block<T, D>(L, kv, i % r.kv_x, i / r.kv_x, sh.pack);
}

template <typename T, int D, int NT, bool Q_ROLE>
int launch_prepare(const Layer& L, const PackKv* kv, const PackQ* q, const Bounds* bn, const Order* od, const KeyList* kl,
                   hipStream_t st) {
  Roles r{};
  const int BH = L.B * L.Hq;
  if (od) r.order = (int)cdiv(sched_cap(od->BH, od->N, od->tile_m), (size_t)(NT / kRankLanes));
  r.keys = kl ? 1 : 0;
  if (bn) {
    r.bounds_x = cdiv(bn->kfirst ? std::max(L.N, bn->npad) : L.N, NT);
    r.bounds = r.bounds_x * BH * (bn->kfirst ? 3 : bn->X ? 2 : 1);
  }
  if (q) {
    r.q_x = q->nqpad / 64;
    r.q = r.q_x * BH;
  }
  long long blocks = (long long)r.order + r.keys + r.bounds + r.q;
  if (kv) {
    const int outputs = (kv->Kn != nullptr) + (kv->Vn != nullptr) + (kv->Kt != nullptr) + (kv->Vt != nullptr);
    if (sizeof(T) == 2 && (outputs * kOutThreads > NT || (kv->Kt && kv->Vt)))
      OMNI_FAIL(OMNI_ERR_UNSUPPORTED, "pack: more copies than the workgroup has room for");
    r.kv_x = kv->npad / kTileN;
    blocks += (long long)r.kv_x * L.B * (kv->per_q_head ? L.Hq : L.Hkv);
  }
  if (blocks >= 0xffffffffll / NT) OMNI_FAIL(OMNI_ERR_UNSUPPORTED, "pack: too many tiles");
  ProfScope prof__(kv || q ? kProfPack : kProfClear, st);
  hipLaunchKernelGGL((prepare_kernel<T, D, NT, Q_ROLE>), dim3((unsigned)blocks), dim3(NT), 0, st, L, r, kv ? *kv : PackKv{},
                     q ? *q : PackQ{}, bn ? *bn : Bounds{}, od ? *od : Order{}, kl ? *kl : KeyList{});
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

// Threads of a workgroup: what the tiles' copies need side by side.
template <typename T, int D>
int launch_prepare(const Layer& L, const PackKv* kv, const PackQ* q, const Bounds* bn, const Order* od, const KeyList* kl,
                   bool backward, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    if (backward) return launch_prepare<T, D, kThreads + 2 * D, true>(L, kv, q, bn, od, kl, st);
  } else if (backward) {
    return launch_prepare<T, D, kThreads, true>(L, kv, q, bn, od, kl, st);
  }
  return launch_prepare<T, D, kThreads, false>(L, kv, q, bn, od, kl, st);
}

}  // namespace

int run_prepare(const Layer& L, int dtype, bool backward, const PackKv* kv, const PackQ* q, const Bounds* bn, const Order* od,
                const KeyList* kl, hipStream_t st) {
  if (dtype == OMNI_BF16) {
    if (L.D == 128) return launch_prepare<u16, 128>(L, kv, q, bn, od, kl, backward, st);
    return launch_prepare<u16, 64>(L, kv, q, bn, od, kl, backward, st);
  }
  if (L.D == 128) return launch_prepare<float, 128>(L, kv, q, bn, od, kl, backward, st);
  return launch_prepare<float, 64>(L, kv, q, bn, od, kl, backward, st);
}

}  // namespace omni
