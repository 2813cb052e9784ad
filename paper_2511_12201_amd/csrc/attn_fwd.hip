// FlashAttention-style forward over kept queries and packed (gathered) keys:
// omni_sparse_attn_fwd and the dense baseline omni_dense_attn_fwd (paper Sec.
// "Preliminary", attention equation, restricted by the masks M^Q, M^K, M^V).
//
// Design for gfx950:
//  * A pack pass (pack.hip) gathers each head's selected K rows into a dense
//    buffer in fragment order (the long fp32 kernel: rows as they are) and its V rows into the exact operand order the matrix cores need
//    (below; rows as they are for the long fp32 kernel), zero-padding to whole
//    64-key tiles.  The dense baseline runs the same pack
//    with identity indices per KV head.  The main loop is then free of gathers.
//  * Both GEMMs are computed transposed, S^T = K Q^T and O^T = V^T P^T, with
//    32x32 MFMA tiles.  Each lane then owns one query column: the softmax row
//    statistics are per-lane scalars (one exchange with the partner lane that
//    holds the other half of the keys), and the S^T accumulator registers are
//    already in the B-operand order of the second GEMM, so P never moves.
//  * V is packed so that the A operand of O^T = V^T P^T is one 16-byte LDS read:
//    [16-key group][d / 32][half h][d % 32][8 keys], key(group,h,j) = 16 group + 8 (j/4) + 4 h + j%4,
//    which is the order in which the S^T accumulators hold the keys.
//  * bf16 inputs, second product in f16: S^T = K Q^T runs on the bf16 matrix cores; the weights are rounded to
//    f16 (11 significant bits against bf16's 8, same matrix-core rate) and multiplied with V converted to f16 by
//    the pack pass (exact for magnitudes in [2^-14, 65504]; beyond that V saturates, below it keeps 3e-8 absolute).
//    The normaliser is the sum of the weights as rounded, so a row that one key dominates returns that key's V row
//    whatever value the weights are taken against, and the log-sum-exp is off by at most 2^-11 relative in the sum.
//  * bf16 (attn_fwd_bf16_kernel, the measured path): 512 threads = 8 wavefronts x
//    32 query rows per work item of 256 kept queries; 64-key K/V tiles go from
//    memory straight into a ring of four LDS stages (global_load_lds, hand-placed
//    s_waitcnt), one barrier per tile; inside a wavefront the softmax of tile t
//    runs under the MFMAs of tile t+1.  Work items come from a persistent,
//    longest-first work list with one queue per XCD (sched_dev.h); causal masks are
//    position compares against per-query visible-prefix counts (bounds_block, sched_dev.h).
//    Short sequences go through attn_fwd_split_kernel: 32-row items, key tiles dealt to the wavefronts.
//  * fp32 inputs (the accuracy path of the 1e-4 parity cases): the fp32 32x32x2 MFMA.  Short sequences
//    (attn_fwd_f32_kernel) have the division of labour of the split kernel, long ones (attn_fwd_f32_long_kernel) 128-row
//    work items with the tiles in LDS.

#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "sched.h"

namespace omni {

namespace {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// ------------------------------------------------------------------ attention

struct FwdParams {
  const void* Q;
  void* O;
  float* lse;
  Layer L;
  const int* q_idx;     // [B*Hq, N] kept query rows, ascending; nullptr: all rows
  const int* q_cnt;     // [B*Hq]; nullptr: N
  const void* Kp;       // packed keys  [BHx, npad, D]: row-major, or in fragment order (short sequences)
  const void* Vp;       // packed values: k-packed, or row-major (fp32 on long sequences)
  const int* budget;    // [B] (or [B,Hq] when L.bph) number of packed keys (device); nullptr: N
  int b_cap;
  int npad;
  int per_q_head;       // packed buffers per query head (sparse) or per KV head (dense)
  int identity_keys;    // slot p is token p: causal bounds by arithmetic (dense baseline)
  const int* qvis;      // [B*Hq, N] visible packed keys per kept-query position; nullptr with identity_keys
  int* sched;           // work list (sched.h)
  size_t order_off;     // where its hand-out order starts
  const int* tile_map;  // in-place variant: [B*Hq, tile_stride] tile of the packed K/V that tile t of a head's key list is
  int tile_stride;
};

// ------------------------------------------------------------------ bf16 fast path
//
// 512 threads = 8 wavefronts x 32 query rows (256-row work items, one workgroup per CU).
// K/V tiles go from global memory straight into LDS (global_load_lds, no VGPR staging) into a
// ring of kStages buffers, so up to kStages - 1 tiles are in flight while one is computed and a
// single barrier per tile is enough.  The loads are inline assembly with hand-placed
// s_waitcnt vmcnt(n): the compiler would wait for *every* outstanding LDS-DMA load before the
// first LDS read, which collapses the ring to one tile of prefetch.
// A wavefront's LDS-DMA instruction writes 64 x 16 contiguous bytes, and a fragment is 64 x 16 bytes lane by lane: the
// packs lay K out in fragment order and V k-packed, a fragment a contiguous kilobyte, so the tile needs no swizzle, its
// reads meet no bank twice and one address register serves it all.

constexpr int kFastWaves = 8;
constexpr int kFastThreads = kFastWaves * 64;
constexpr int kFastTileM = kFastWaves * 32;
constexpr int kStages = 4;
constexpr int kMaxMapTiles = 2048;                   // key tiles of one head in the in-place variant (128k tokens)

// TILEMAP: the key list of a head is a sequence of whole 64-key tiles of the KV head's (ungathered) K/V -- the
// block-granular selection -- and tile t of the list is read in place, at tile p.tile_map[head][t].
template <int D, bool TILEMAP>
__global__ __launch_bounds__(kFastThreads, 2) void attn_fwd_bf16_kernel(FwdParams p) {
  typedef u16 T;
  constexpr int kKBytes = kTileN * D * 2;
  constexpr int kStageBytes = 2 * kKBytes;           // K tile then V tile
  constexpr int LPH = kKBytes / 1024 / kFastWaves;   // load instructions per operand per wavefront per tile
  constexpr int LPT = 2 * LPH;
  static_assert(LPH >= 1, "tile too small for the copy scheme");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kStages * kStageBytes];
  __shared__ int sBound[2];
  __shared__ int sItem;
  __shared__ int sTileMap[TILEMAP ? kMaxMapTiles : 1];

  const Layer& L = p.L;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int lane_b = lane * 16;                                // copies and fragment reads: 16 bytes a lane, in lane order

  for (;;) {
  __syncthreads();
  if (threadIdx.x == 0) sItem = sched_next(p.sched);
  __syncthreads();
  const int item = __builtin_amdgcn_readfirstlane(sItem);   // wave-uniform, and known to be: tile bases stay in SGPRs
  if (item < 0) break;
  int bh, tq;
  sched_decode(p.sched, p.order_off, item, bh, tq);
  bh = __builtin_amdgcn_readfirstlane(bh);
  tq = __builtin_amdgcn_readfirstlane(tq);
  const int b = bh / L.Hq, i = bh % L.Hq, g = i / L.G;
  const int nq = p.q_cnt ? p.q_cnt[bh] : L.N;
  const int nkeys = p.budget ? min(p.budget[budget_slot(L.bph, b, bh)], p.b_cap) : L.N;
  const int bhx = p.per_q_head ? bh : b * L.Hkv + g;
  const int* qlist = p.q_idx ? p.q_idx + (long long)bh * L.N : nullptr;

  const int pos_first = tq * kFastTileM, pos_last = min(pos_first + kFastTileM, nq) - 1;
  const int* qvis = p.qvis + (long long)bh * L.N;          // not read for the dense baseline
  // visible prefix length of the packed key list for a kept-query position
  auto visible = [&](int pos, int row) {
    if (!L.causal) return nkeys;
    if (p.identity_keys) return min(row + 1, nkeys);
    return qvis[pos];
  };
  if (threadIdx.x == 0 || threadIdx.x == 64) {
    const int which = threadIdx.x ? 1 : 0;
    const int pos = which ? pos_last : pos_first;
    sBound[which] = visible(pos, qlist ? qlist[pos] : pos);
  }
  __syncthreads();
  const int n_full_tiles = sBound[0] / kTileN;
  const int ntiles = cdiv(sBound[1], kTileN);
  if constexpr (TILEMAP) {                                     // this item's share of the head's tile map
    const int* tm = p.tile_map + (long long)bh * p.tile_stride;
    for (int t = threadIdx.x; t < ntiles; t += kFastThreads) sTileMap[t] = tm[t];
    __syncthreads();
  }

  const int qpos = pos_first + wave * 32 + ln;
  const bool qvalid = qpos < nq;
  const int qpos_c = min(qpos, nq - 1);
  const int qrow = qlist ? qlist[qpos_c] : qpos_c;
  const int qvisible = visible(qpos_c, qrow) - 4 * h;          // compared with key positions that leave out 4 * h
  const T* qptr = static_cast<const T*>(p.Q) + b * L.qs[0] + i * L.qs[1] + (long long)qrow * L.qs[2];
  bf16x8 qf[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qptr + ks * 16 + h * 8);
  // Make the compiler finish these loads here.  Otherwise it places their s_waitcnt vmcnt at the first
  // use inside the tile loop, where it would also drain the K/V prefetch ring on every iteration.
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) asm volatile("" : "+v"(qf[ks]));

  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const T* kp = static_cast<const T*>(p.Kp) + (long long)bhx * p.npad * D;
  const T* vp = static_cast<const T*>(p.Vp) + (long long)bhx * p.npad * D;

  // one load instruction of tile t: part < LPH is a K part, the rest are V parts
  auto issue_part = [&](int t, int part) {
    const unsigned dst = lds_base + (unsigned)(t % kStages) * kStageBytes;
    // where tile t of the key list lives (wave-uniform: the tile base stays in scalar registers)
    const int src = TILEMAP ? __builtin_amdgcn_readfirstlane(sTileMap[t]) : t;
    if (part < LPH) {
      const int at = part * kFastWaves + wave;
      gload_lds16(kp + (long long)src * kTileN * D + at * 512, lane_b, dst + at * 1024);
    } else {
      const int at = (part - LPH) * kFastWaves + wave;
      gload_lds16(vp + (long long)src * kTileN * D + at * 512, lane_b, dst + kKBytes + at * 1024);
    }
  };
  auto issue_tile = [&](int t) {
#pragma unroll
    for (int j = 0; j < LPT; ++j) issue_part(t, j);
  };

  // Software pipeline over key tiles.  While the matrix cores compute S(t+1)^T = K(t+1) . Q^T the
  // same wavefront turns S(t) into P(t) on the vector ALU (exp2, f16 pack, row sum); while they
  // accumulate O^T += V(t)^T . P(t)^T it scans S(t+1) for the running maximum (in the steps that follow
  // it; see `step`).  Each MFMA is followed
  // in program order by its share of the vector work and a scheduling fence, so the hardware always
  // has independent vector instructions to issue under a running MFMA.  Without this the two
  // wavefronts of a SIMD, which the per-tile barrier keeps in step, are in their softmax phases at
  // the same time and the matrix cores idle for that long.
  constexpr int NQK = 2 * (D / 16);          // MFMAs of one S tile: 2 key blocks x D/16 k-steps
  constexpr int NPV = 4 * (D / 32);          // MFMAs of one P.V tile: 4 key steps x D/32 row blocks
  constexpr int NB = D / 32;
  constexpr int kAhead = 2;                  // fragment reads run this many MFMAs ahead
  static_assert(32 % NQK == 0 && 32 % NPV == 0 && 16 % NPV == 0, "chunking of the vector work");
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  auto kfrag = [&](const unsigned char* sk, int c) {
    const int kb = c % 2, ks = c / 2;
    return *reinterpret_cast<const bf16x8*>(sk + lane_b + (kb * (D / 16) + ks) * 1024);
  };
  auto vfrag = [&](const unsigned char* sv, int c) {
    return *reinterpret_cast<const f16x8*>(sv + lane_b + c * 1024);
  };

  // S^T of tile t alone (first tile of an item)
  auto qk_only = [&](f32x16 (&sn)[2], int t) {
    const unsigned char* sk = smem + (t % kStages) * kStageBytes;
    bf16x8 kf[kAhead];
#pragma unroll
    for (int c = 0; c < kAhead; ++c) kf[c] = kfrag(sk, c);
#pragma unroll
    for (int c = 0; c < NQK; ++c) {
      const int kb = c % 2, ks = c / 2;
      __builtin_amdgcn_sched_barrier(0);
      sn[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c % kAhead], qf[ks], ks == 0 ? zero16 : sn[kb], 0, 0, 0);
      if (c + kAhead < NQK) kf[c % kAhead] = kfrag(sk, c + kAhead);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // Reference value of the softmax from a finished S tile.  m_run is the value the weights are taken against, not
  // the exact running maximum: it moves (and the accumulators are rescaled) only when some row of the wavefront
  // exceeds it by more than kRescaleSlack in the exponent, so a weight is at most 2^kRescaleSlack and the rescale
  // is rare.  Output and log-sum-exp do not depend on the reference value beyond rounding.
  float mc = 0.f;                              // (reference value, 0 if none yet) * c2
  constexpr float kRescaleSlack = 6.0f;
  auto update_max = [&](float mloc) {
    mloc = pair_max(mloc);
    if (__any(mloc > m_run + kRescaleSlack / c2)) {
      const float m_new = fmaxf(m_run, mloc);
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = fast_exp2((m_run - m_ref) * c2);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m_run = m_new;
      mc = m_ref * c2;
    }
  };
  auto mask_tile = [&](f32x16 (&sn)[2], int t) {
    const int rel = qvisible - t * kTileN;     // keys of this tile at positions >= rel are hidden (pad rows too)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (kb * 32 + 8 * q4 + e >= rel) sn[kb][q4 * 4 + e] = -INFINITY;   // register r holds key 8 (r/4) + 4 h + r%4
    float mloc = sn[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; r += 2) mloc = fmaxf(fmaxf(sn[kb][r], sn[kb][r + 1]), mloc);
    return mloc;
  };

  // Steps that do not follow the maximum (below) call this when a weight left the safe range: the reference value
  // moves to the maximum of the tile at hand, the accumulators are rescaled, and the tile's weights are formed again.
  union PFrag { f16x8 v[4]; f16x2 h[16]; };
  // acc + both halves of pk, one instruction each: the sum of the weights exactly as the matrix cores get them
  auto add_halves = [](float acc, f16x2 pk) {
    asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "+v"(acc) : "v"(pk));
    asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(acc) : "v"(pk));
    return acc;
  };
  auto refit = [&](const f32x16 (&sc)[2], PFrag& pf, float& lsum) {
    float mloc = sc[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; r += 2) mloc = fmaxf(fmaxf(sc[kb][r], sc[kb][r + 1]), mloc);
    mloc = pair_max(mloc);
    const float m_new = fmaxf(m_run, mloc);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = fast_exp2((m_run - m_ref) * c2);
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    m_run = m_new;
    mc = m_ref * c2;
    lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 32; r += 2) {
      f32x2 pv;
      pv[0] = fast_exp2(fmaf(sc[r / 16][r % 16], c2, -mc));
      pv[1] = fast_exp2(fmaf(sc[r / 16][r % 16 + 1], c2, -mc));
      const f16x2 pk = __builtin_convertvector(pv, f16x2);
      pf.h[r / 2] = pk;
      lsum = add_halves(lsum, pk);
    }
  };

  // One pipeline step: P(t) from sc, O += V(t) P(t); if there is a tile t+1: S(t+1) into sn and its maximum.
  // `steady` steps are the ones with t + 3 < ntiles: they always have a next tile and always prefetch,
  // so the step is straight-line code and the fences keep the interleaving as written.
  // `follow` steps scan S(t+1) for its maximum and move the reference value by the slack rule.  Once every row of
  // the wavefront has a reference value (a finite one: it has seen a key), the steady steps stop following: a
  // reference value that is the maximum of some of the row's logits can only be too low, never too high, so a weight
  // that underflows is below 2^-126 of the row's largest and does not matter, and one that grows past kHuge shows in
  // the tile's sum of weights, which is there anyway -- then refit() moves the reference.  That takes the maximum
  // scan and its bookkeeping (a sixth of the step's vector instructions) out of the loop.
  constexpr float kHuge = 16384.f;                 // 2^14: a weight stays inside the f16 range
  auto step = [&](auto steady, auto follows, f32x16 (&sc)[2], f32x16 (&sn)[2], int t) {
    constexpr bool kSteady = decltype(steady)::value;
    constexpr bool kFollow = decltype(follows)::value;
    const bool has_next = kSteady || t + 1 < ntiles;
    const int pre = (kSteady || t + 3 < ntiles) ? t + 3 : -1;
    const unsigned char* sk = smem + ((t + 1) % kStages) * kStageBytes;
    const unsigned char* sv = smem + (t % kStages) * kStageBytes + kKBytes;
    PFrag pf;
    float lsum = 0.f;
    f16x8 vf[kAhead];
    constexpr int EQ = 32 / NQK;             // S elements turned into P per QK MFMA
    auto softmax_chunk = [&](int c) {
#pragma unroll
      for (int e = 0; e < EQ; e += 2) {
        const int r = c * EQ + e;
        f32x2 pv;
        pv[0] = fast_exp2(fmaf(sc[r / 16][r % 16], c2, -mc));
        pv[1] = fast_exp2(fmaf(sc[r / 16][r % 16 + 1], c2, -mc));
        const f16x2 pk = __builtin_convertvector(pv, f16x2);
        pf.h[r / 2] = pk;
        lsum = add_halves(lsum, pk);           // the weights as rounded: numerator and normaliser agree
      }
    };
    if (has_next) {
      if (kSteady || t + 2 < ntiles) wait_vmcnt<LPT>();   // this wavefront's share of tile t+1 has landed
      else wait_vmcnt<0>();
      __syncthreads();                        // ... and everyone else's; tile t-1 is retired
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 kf[kAhead];
#pragma unroll
      for (int c = 0; c < kAhead; ++c) kf[c] = kfrag(sk, c);
#pragma unroll
      for (int c = 0; c < NQK; ++c) {
        const int kb = c % 2, ks = c / 2;
        __builtin_amdgcn_sched_barrier(0);
        sn[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c % kAhead], qf[ks], ks == 0 ? zero16 : sn[kb], 0, 0, 0);
        if (c + kAhead < NQK) kf[c % kAhead] = kfrag(sk, c + kAhead);
        else vf[c + kAhead - NQK] = vfrag(sv, c + kAhead - NQK);
        softmax_chunk(c);
        if (c * LPH % NQK == 0 && (kSteady || pre >= 0)) issue_part(pre, c * LPH / NQK);
      }
    } else {
#pragma unroll
      for (int c = 0; c < kAhead; ++c) vf[c] = vfrag(sv, c);
#pragma unroll
      for (int c = 0; c < NQK; ++c) softmax_chunk(c);
    }
    // (also in the following steps: the first one after a stretch that did not follow forms its weights against
    // the reference value that stretch left behind)
    if (__any(lsum > kHuge)) refit(sc, pf, lsum);
    l_run += lsum;
    __builtin_amdgcn_s_setprio(0);
    float mloc = -INFINITY;
    constexpr int EV = 32 / NPV;             // S(t+1) elements scanned per P.V MFMA
#pragma unroll
    for (int c = 0; c < NPV; ++c) {
      const int t16 = c / NB, db = c % NB;
      __builtin_amdgcn_sched_barrier(0);
      o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[c % kAhead], pf.v[t16], o[db], 0, 0, 0);
      if (c + kAhead < NPV) vf[c % kAhead] = vfrag(sv, c + kAhead);
      if constexpr (kFollow) {
#pragma unroll
        for (int e = 0; e < EV; e += 2) {
          const int r = c * EV + e;
          mloc = fmaxf(fmaxf(sn[r / 16][r % 16], sn[r / 16][r % 16 + 1]), mloc);
        }
      }
      if (c * LPH % NPV == 0 && (kSteady || pre >= 0)) issue_part(pre, LPH + c * LPH / NPV);
    }
    __builtin_amdgcn_sched_barrier(0);
    // The mixed MFMA + vector block and the bookkeeping run at raised priority, the pure MFMA block at the
    // base one: the wavefront with vector work to issue wins the arbiter, the other one's MFMAs fill in.
    __builtin_amdgcn_s_setprio(1);
    if (has_next) {
      if (t + 1 >= n_full_tiles) mloc = mask_tile(sn, t + 1);
      if constexpr (kFollow) update_max(mloc);
    }
  };

  // Ring of kStages buffers, one barrier per tile.  At the top of step t the tiles up to t+2 have been
  // issued; after its barrier everyone is done with tile t-1, whose buffer takes tile t+3.  The loads of
  // tile t+3 are spread over the MFMAs of the step instead of being issued in one burst: the CU moves
  // about 64 bytes per clock from memory into LDS, so a burst of all eight wavefronts backs the queue
  // up and stalls the issuing wavefronts for hundreds of cycles.
  static_assert(kStages == 4, "the wait counts assume this ring depth");
  if (ntiles > 0) {
    f32x16 sa[2], sb[2];
    sb[0] = zero16;
    sb[1] = zero16;
    wait_vmcnt<0>();                        // nothing of the previous item (its output stores) is counted below
    issue_tile(0);
    if (ntiles > 1) issue_tile(1);
    if (ntiles > 2) issue_tile(2);
    if (ntiles > 2) wait_vmcnt<2 * LPT>();
    else if (ntiles > 1) wait_vmcnt<LPT>();
    else wait_vmcnt<0>();
    __syncthreads();
    qk_only(sa, 0);
    {
      float mloc;
      if (0 >= n_full_tiles) {
        mloc = mask_tile(sa, 0);
      } else {
        mloc = sa[0][0];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; r += 2) mloc = fmaxf(fmaxf(sa[kb][r], sa[kb][r + 1]), mloc);
      }
      update_max(mloc);
    }
    int t = 0;
    for (; t + 4 < ntiles && __any(m_run == -INFINITY); t += 2) {   // some row has not seen a key yet
      step(std::true_type{}, std::true_type{}, sa, sb, t);
      step(std::true_type{}, std::true_type{}, sb, sa, t + 1);
    }
    for (; t + 4 < ntiles; t += 2) {
      step(std::true_type{}, std::false_type{}, sa, sb, t);
      step(std::true_type{}, std::false_type{}, sb, sa, t + 1);
    }
    for (; t < ntiles; t += 2) {
      step(std::false_type{}, std::true_type{}, sa, sb, t);
      if (t + 1 < ntiles) step(std::false_type{}, std::true_type{}, sb, sa, t + 1);
    }
  }

  const float l_tot = pair_sum(l_run);
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  if (qvalid) {
    T* optr = static_cast<T*>(p.O) + b * L.qs[0] + i * L.qs[1] + (long long)qrow * L.qs[2];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d = db * 32 + 8 * q4 + 4 * h;
        uint2 w;
        w.x = pack_bf16x2(o[db][q4 * 4 + 0] * inv, o[db][q4 * 4 + 1] * inv);
        w.y = pack_bf16x2(o[db][q4 * 4 + 2] * inv, o[db][q4 * 4 + 3] * inv);
        *reinterpret_cast<uint2*>(optr + d) = w;
      }
    if (h == 0)
      p.lse[(long long)bh * L.N + qrow] = l_tot > 0.f ? (m_run * c2 + log2f(l_tot)) * kLn2 : -INFINITY;
  }
  }  // work-item loop
}

// ------------------------------------------------------------------ bf16, short sequences
//
// The kernel above needs long items: 256 rows keep its eight wavefronts busy for 2 us a tile, and a launch of a few dozen
// items leaves most CUs idle while each walks its tiles one after the other (36 us for 60 items of at most 10 tiles).
// Here an item is 32 kept queries and its four wavefronts share the key tiles, every fourth tile each, with softmax states
// of their own that are merged at the end: eight times the items, a quarter of the chain.  No staging and no barrier in
// the loop: both operands lie in fragment order in memory, so that a fragment is one contiguous kilobyte per wavefront, and
// the next K tile is loaded under the softmax and the second product.  Every item reads its whole K/V prefix through the
// CU's L1 (64 bytes a clock), which is what bounds it: an item of the kernel above shares those bytes between 256 rows.
constexpr int kSplitWaves = 4;
constexpr int kSplitThreads = kSplitWaves * 64;
constexpr int kSplitRows = 32;

// grid: cdiv(N, kSplitRows) * B*Hq, heads fastest; a head's last rows, which see the most keys, first
template <int D, bool TILEMAP>
__global__ __launch_bounds__(kSplitThreads, 2) void attn_fwd_split_kernel(FwdParams p) {
  typedef u16 T;
  constexpr int CH = D / 8, KS = D / 16, NB = D / 32;
  constexpr int OP = D + 4;                          // floats between rows of the merge buffer
  __shared__ __attribute__((aligned(16))) unsigned char sQ[kSplitRows * D * 2];
  __shared__ __attribute__((aligned(16))) float sO[kSplitWaves][kSplitRows][OP];
  __shared__ float sM[kSplitWaves][kSplitRows], sL[kSplitWaves][kSplitRows];
  const Layer& L = p.L;
  const int BH = L.B * L.Hq, bh = blockIdx.x % BH, b = bh / L.Hq, i = bh % L.Hq, g = i / L.G;
  const int nq = p.q_cnt[bh];
  const int tq = cdiv(nq, kSplitRows) - 1 - (int)(blockIdx.x / BH);
  if (tq < 0) return;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const int* qlist = p.q_idx + (long long)bh * L.N;
  const int* qvis = p.qvis + (long long)bh * L.N;
  const int pos_first = tq * kSplitRows, pos_last = min(pos_first + kSplitRows, nq) - 1;
  const int n_full_tiles = qvis[pos_first] / kTileN, ntiles = cdiv(qvis[pos_last], kTileN);
  const int pos_c = min(pos_first + ln, nq - 1);
  const int qvisible = qvis[pos_c] - 4 * h;
  const T* qhead = static_cast<const T*>(p.Q) + b * L.qs[0] + i * L.qs[1];
#pragma unroll
  for (int c = threadIdx.x; c < kSplitRows * CH; c += kSplitThreads) {
    const int row = c / CH, chunk = c % CH;
    const u32x4 v = *reinterpret_cast<const u32x4*>(qhead + (long long)qlist[min(pos_first + row, nq - 1)] * L.qs[2] + chunk * 8);
    *reinterpret_cast<u32x4*>(sQ + (row * CH + (chunk ^ (row % CH))) * 16) = v;
  }
  const int bhx = p.per_q_head ? bh : b * L.Hkv + g;
  const unsigned char* kp = static_cast<const unsigned char*>(p.Kp) + (long long)bhx * p.npad * D * 2 + lane * 16;
  const unsigned char* vp = static_cast<const unsigned char*>(p.Vp) + (long long)bhx * p.npad * D * 2 + lane * 16;
  const int* tile_map = TILEMAP ? p.tile_map + (long long)bh * p.tile_stride : nullptr;
  auto tile_bytes = [&](int t) {
    const int src = TILEMAP ? __builtin_amdgcn_readfirstlane(tile_map[t]) : t;
    return (long long)src * (kTileN * D * 2);
  };
  bf16x8 kf[2][KS];
  auto load_k = [&](int t) {
    const unsigned char* k = kp + tile_bytes(t);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[kb][ks] = *reinterpret_cast<const bf16x8*>(k + (kb * KS + ks) * 1024);
  };
  f32x16 o[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  if (wave < ntiles) load_k(wave);
  __syncthreads();
  for (int t = wave; t < ntiles; t += kSplitWaves) {
    f16x8 vf[2][NB];
    const unsigned char* v = vp + tile_bytes(t);
    auto load_v = [&](int half) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int db = 0; db < NB; ++db) vf[u][db] = *reinterpret_cast<const f16x8*>(v + ((half * 2 + u) * NB + db) * 1024);
    };
    load_v(0);
    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 qf = *reinterpret_cast<const bf16x8*>(sQ + (ln * CH + ((2 * ks + h) ^ (ln % CH))) * 16);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][ks], qf, s[kb], 0, 0, 0);
    }
    if (t + kSplitWaves < ntiles) load_k(t + kSplitWaves);
    if (t >= n_full_tiles) {
      const int rel = qvisible - t * kTileN;         // keys of this tile at positions >= rel are hidden (pad rows too)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb * 32 + 8 * (r >> 2) + (r & 3) >= rel) s[kb][r] = -INFINITY;
    }
    float m = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, s[kb][r]);
    m = fmaxf(m_run, pair_max(m));
    const float m_ref = m == -INFINITY ? 0.f : m, mc = m_ref * c2;
    if (__any(m > m_run)) {
      const float alpha = fast_exp2((m_run - m_ref) * c2);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m_run = m;
    }
    union { f16x8 v[4]; f16x2 h2[16]; } pf;
#pragma unroll
    for (int r = 0; r < 32; r += 2) {
      f32x2 pv;
      pv[0] = fast_exp2(fmaf(s[r / 16][r % 16], c2, -mc));
      pv[1] = fast_exp2(fmaf(s[r / 16][r % 16 + 1], c2, -mc));
      const f16x2 pk = __builtin_convertvector(pv, f16x2);
      pf.h2[r / 2] = pk;
      l_run += (float)pk[0] + (float)pk[1];          // the weights as rounded: numerator and normaliser agree
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int db = 0; db < NB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[u][db], pf.v[half * 2 + u], o[db], 0, 0, 0);
      if (half == 0) load_v(1);
    }
  }

  // merge the wavefronts in their order
  const float l_own = pair_sum(l_run);
  if (h == 0) {
    sM[wave][ln] = m_run;
    sL[wave][ln] = l_own;
  }
  __syncthreads();
  float top = sM[0][ln];
#pragma unroll
  for (int w = 1; w < kSplitWaves; ++w) top = fmaxf(top, sM[w][ln]);
  const float ref = top == -INFINITY ? 0.f : top;
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < kSplitWaves; ++w) total += sL[w][ln] * fast_exp2((sM[w][ln] - ref) * c2);
  const float mine = total > 0.f ? fast_exp2((m_run - ref) * c2) / total : 0.f;
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 v = {o[db][q4 * 4] * mine, o[db][q4 * 4 + 1] * mine, o[db][q4 * 4 + 2] * mine, o[db][q4 * 4 + 3] * mine};
      *reinterpret_cast<f32x4*>(&sO[wave][ln][db * 32 + 8 * q4 + 4 * h]) = v;
    }
  if (threadIdx.x < kSplitRows && pos_first + (int)threadIdx.x < nq)
    p.lse[(long long)bh * L.N + qlist[pos_first + threadIdx.x]] = total > 0.f ? (top * c2 + log2f(total)) * kLn2 : -INFINITY;
  __syncthreads();
  T* ohead = static_cast<T*>(p.O) + b * L.qs[0] + i * L.qs[1];
#pragma unroll
  for (int c = threadIdx.x; c < kSplitRows * CH; c += kSplitThreads) {
    const int row = c / CH, d = c % CH * 8;
    if (pos_first + row >= nq) continue;
    f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      x += *reinterpret_cast<const f32x4*>(&sO[w][row][d]);
      y += *reinterpret_cast<const f32x4*>(&sO[w][row][d + 4]);
    }
    const u32x4 out = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    *reinterpret_cast<u32x4*>(ohead + (long long)qlist[pos_first + row] * L.qs[2] + d) = out;
  }
}

// ------------------------------------------------------------------ fp32
//
// The same division of labour on the fp32 matrix cores (32x32x2, one element per lane and step): an item is 32 query rows,
// its four wavefronts share the 64-key tiles, both operands come straight from memory, four elements of a lane with one
// 16-byte read.  Bound by those matrix instructions (64 cycles each, 128 of them per tile at d = 64: 4 us), whose chain
// per item this cuts to a quarter; tiles staged through LDS for four wavefronts of 32 rows, without overlap, took 62 us on
// 24 items of 1k tokens, this takes 18.  No list, longest items first: the dispatcher balances.
template <int D>
__global__ __launch_bounds__(kSplitThreads, D == 64 ? 2 : 1) void attn_fwd_f32_kernel(FwdParams p) {
  constexpr int CH = D / 4, KS = D / 8, NB = D / 32;
  constexpr int OP = D + 4;                          // floats between rows of the merge buffer
  __shared__ __attribute__((aligned(16))) float sO[kSplitWaves][kSplitRows][OP];
  __shared__ float sM[kSplitWaves][kSplitRows], sL[kSplitWaves][kSplitRows];
  const Layer& L = p.L;
  const int BH = L.B * L.Hq, bh = blockIdx.x % BH, b = bh / L.Hq, i = bh % L.Hq, g = i / L.G;
  const int nq = p.q_cnt ? p.q_cnt[bh] : L.N;
  const int tq = cdiv(nq, kSplitRows) - 1 - (int)(blockIdx.x / BH);
  if (tq < 0) return;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  const int* qlist = p.q_idx ? p.q_idx + (long long)bh * L.N : nullptr;       // null: all rows, all keys (dense baseline)
  const int* qvis = p.qvis ? p.qvis + (long long)bh * L.N : nullptr;
  auto row_of = [&](int pos) { return qlist ? qlist[pos] : pos; };
  auto visible = [&](int pos) { return qvis ? qvis[pos] : (L.causal ? pos + 1 : L.N); };
  const int pos_first = tq * kSplitRows, pos_last = min(pos_first + kSplitRows, nq) - 1;
  const int n_full_tiles = visible(pos_first) / kTileN, ntiles = cdiv(visible(pos_last), kTileN);
  const int pos_c = min(pos_first + ln, nq - 1);
  const int qvisible = visible(pos_c) - 4 * h;
  const float* qhead = static_cast<const float*>(p.Q) + b * L.qs[0] + i * L.qs[1];
  const float* qrow = qhead + (long long)row_of(pos_c) * L.qs[2];
  f32x4 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const f32x4*>(qrow + ks * 8 + h * 4);
  const int bhx = p.per_q_head ? bh : b * L.Hkv + g;
  const float* kp = static_cast<const float*>(p.Kp) + (long long)bhx * p.npad * D + lane * 4;
  const float* vp = static_cast<const float*>(p.Vp) + (long long)bhx * p.npad * D + lane * 4;
  f32x4 kf[2][KS];
  auto load_k = [&](int t) {
    const float* k = kp + (long long)t * kTileN * D;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[kb][ks] = *reinterpret_cast<const f32x4*>(k + (kb * KS + ks) * 256);
  };
  f32x16 o[NB];
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  if (wave < ntiles) load_k(wave);
  for (int t = wave; t < ntiles; t += kSplitWaves) {
    f32x4 vf[2][4][NB];
    const float* v = vp + (long long)t * kTileN * D;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int db = 0; db < NB; ++db) vf[kb][q4][db] = *reinterpret_cast<const f32x4*>(v + ((kb * 4 + q4) * NB + db) * 256);
    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) s[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[kb][ks][e], qf[ks][e], s[kb], 0, 0, 0);
    if (t + kSplitWaves < ntiles) load_k(t + kSplitWaves);
    if (t >= n_full_tiles) {
      const int rel = qvisible - t * kTileN;         // keys of this tile at positions >= rel are hidden (pad rows too)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb * 32 + 8 * (r >> 2) + (r & 3) >= rel) s[kb][r] = -INFINITY;
    }
    float m = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, s[kb][r]);
    m = fmaxf(m_run, pair_max(m));
    const float m_ref = m == -INFINITY ? 0.f : m, mc = m_ref * c2;
    if (__any(m > m_run)) {
      const float alpha = fast_exp2((m_run - m_ref) * c2);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m_run = m;
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[kb][r] = fast_exp2(fmaf(s[kb][r], c2, -mc));
        l_run += s[kb][r];
      }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int db = 0; db < NB; ++db)
          o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[kb][r >> 2][db][r & 3], s[kb][r], o[db], 0, 0, 0);
  }

  // merge the wavefronts in their order
  const float l_own = pair_sum(l_run);
  if (h == 0) {
    sM[wave][ln] = m_run;
    sL[wave][ln] = l_own;
  }
  __syncthreads();
  float top = sM[0][ln];
#pragma unroll
  for (int w = 1; w < kSplitWaves; ++w) top = fmaxf(top, sM[w][ln]);
  const float ref = top == -INFINITY ? 0.f : top;
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < kSplitWaves; ++w) total += sL[w][ln] * fast_exp2((sM[w][ln] - ref) * c2);
  const float mine = total > 0.f ? fast_exp2((m_run - ref) * c2) / total : 0.f;
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 v = {o[db][q4 * 4] * mine, o[db][q4 * 4 + 1] * mine, o[db][q4 * 4 + 2] * mine, o[db][q4 * 4 + 3] * mine};
      *reinterpret_cast<f32x4*>(&sO[wave][ln][db * 32 + 8 * q4 + 4 * h]) = v;
    }
  if (threadIdx.x < kSplitRows && pos_first + (int)threadIdx.x < nq)
    p.lse[(long long)bh * L.N + row_of(pos_first + threadIdx.x)] = total > 0.f ? (top * c2 + log2f(total)) * kLn2 : -INFINITY;
  __syncthreads();
  float* ohead = static_cast<float*>(p.O) + b * L.qs[0] + i * L.qs[1];
#pragma unroll
  for (int c = threadIdx.x; c < kSplitRows * CH; c += kSplitThreads) {
    const int row = c / CH, d = c % CH * 4;
    if (pos_first + row >= nq) continue;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) x += *reinterpret_cast<const f32x4*>(&sO[w][row][d]);
    *reinterpret_cast<f32x4*>(ohead + (long long)row_of(pos_first + row) * L.qs[2] + d) = x;
  }
}

// fp32, long sequences: 128-row items from the work list, 32 rows per wavefront, K/V tiles staged row by row through LDS.  An
// item of 32 rows streams its whole K/V prefix for itself, and once the 128-row items fill the chip that is what costs
// (f32_short says where the line lies).
template <int D>
__global__ __launch_bounds__(kThreads, 2) void attn_fwd_f32_long_kernel(FwdParams p) {
  constexpr int KLD = D + 4, VLD = D + 8;            // row pitches of the tiles
  constexpr int CPR = D / 4, kChunks = kTileN * CPR / kThreads;      // 16-byte chunks per row, per thread and operand
  __shared__ __attribute__((aligned(16))) float sK[kTileN * KLD], sV[kTileN * VLD];
  __shared__ int sItem;
  const Layer& L = p.L;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int ln = lane & 31, h = lane >> 5;
  const float c2 = L.scale * kLog2e;
  for (;;) {                                         // persistent: one work item (head, query tile) per iteration
    __syncthreads();                                 // LDS of the previous item is no longer read
    if (threadIdx.x == 0) sItem = sched_next(p.sched, 1);
    __syncthreads();
    const int item = sItem;
    if (item < 0) break;
    int bh, tq;
    sched_decode(p.sched, p.order_off, item, bh, tq);
    const int b = bh / L.Hq, i = bh % L.Hq, g = i / L.G;
    const int nq = p.q_cnt ? p.q_cnt[bh] : L.N;
    const int* qlist = p.q_idx ? p.q_idx + (long long)bh * L.N : nullptr;       // null: all rows, all keys (dense baseline)
    const int* qvis = p.qvis ? p.qvis + (long long)bh * L.N : nullptr;
    auto visible = [&](int pos) { return qvis ? qvis[pos] : (L.causal ? pos + 1 : L.N); };
    const int pos_first = tq * kTileM, pos_last = min(pos_first + kTileM, nq) - 1;
    const int n_full_tiles = visible(pos_first) / kTileN, ntiles = cdiv(visible(pos_last), kTileN);
    const int qpos = pos_first + wave * 32 + ln, qpos_c = min(qpos, nq - 1);
    const int qrow = qlist ? qlist[qpos_c] : qpos_c, qvisible = visible(qpos_c) - 4 * h;
    const long long row_off = b * L.qs[0] + i * L.qs[1] + (long long)qrow * L.qs[2];
    f32x4 qf[D / 8];
#pragma unroll
    for (int ks = 0; ks < D / 8; ++ks)
      qf[ks] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.Q) + row_off + ks * 8 + h * 4);
    f32x16 o[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const long long head = (long long)(p.per_q_head ? bh : b * L.Hkv + g) * p.npad * D;
    const float *kp = static_cast<const float*>(p.Kp) + head, *vp = static_cast<const float*>(p.Vp) + head;
    for (int t = 0; t < ntiles; ++t) {
      __syncthreads();
      u32x4 stK[kChunks], stV[kChunks];
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
        stK[c] = *reinterpret_cast<const u32x4*>(kp + (long long)t * kTileN * D + (threadIdx.x + c * kThreads) * 4);
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
        stV[c] = *reinterpret_cast<const u32x4*>(vp + (long long)t * kTileN * D + (threadIdx.x + c * kThreads) * 4);
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const int ch = threadIdx.x + c * kThreads, row = ch / CPR, col = ch % CPR * 4;
        *reinterpret_cast<u32x4*>(sK + row * KLD + col) = stK[c];
        *reinterpret_cast<u32x4*>(sV + row * VLD + col) = stV[c];
      }
      __syncthreads();
      f32x16 s[2];                                   // S^T tile = K tile . Q^T
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 8; ++ks) {
          const f32x4 kf = *reinterpret_cast<const f32x4*>(sK + (kb * 32 + ln) * KLD + ks * 8 + h * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) s[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[ks][e], s[kb], 0, 0, 0);
        }
      }
      if (t >= n_full_tiles) {
        const int rel = qvisible - t * kTileN;       // keys of this tile at positions >= rel are hidden (pad rows too)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (kb * 32 + 8 * (r >> 2) + (r & 3) >= rel) s[kb][r] = -INFINITY;
      }
      float m = s[0][0];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) m = fmaxf(m, s[kb][r]);
      m = fmaxf(m_run, pair_max(m));
      const float m_ref = m == -INFINITY ? 0.f : m, mc = m_ref * c2;
      if (__any(m > m_run)) {
        const float alpha = fast_exp2((m_run - m_ref) * c2);
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        m_run = m;
      }
      float lsum = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          s[kb][r] = fast_exp2(fmaf(s[kb][r], c2, -mc));
          lsum += s[kb][r];
        }
      l_run += lsum;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)                 // O^T += V^T . P^T
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int slot = kb * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
#pragma unroll
          for (int db = 0; db < D / 32; ++db)
            o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(sV[slot * VLD + db * 32 + ln], s[kb][r], o[db], 0, 0, 0);
        }
    }
    const float l_tot = pair_sum(l_run), inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (qpos < nq) {
      float* out = static_cast<float*>(p.O) + row_off;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x4 w = {o[db][q4 * 4] * inv, o[db][q4 * 4 + 1] * inv, o[db][q4 * 4 + 2] * inv, o[db][q4 * 4 + 3] * inv};
          *reinterpret_cast<f32x4*>(out + db * 32 + 8 * q4 + 4 * h) = w;
        }
      if (h == 0) p.lse[(long long)bh * L.N + qrow] = l_tot > 0.f ? (m_run * c2 + log2f(l_tot)) * kLn2 : -INFINITY;
    }
  }
}

// Which of the two bf16 kernels: the bytes an item streams alone make the split kernel the slower one once the work per
// CU outweighs the length of a chain.  Whole attention call in us, (heads, d) N: split / the other, a third of the
// queries and half of the keys kept: (28, 128) 1072: 30 / 55, 3101: 60 / 83, 4096: 85 / 100, 6000: 134 / 129,
// (28, 64) 4096: 53 / 78, 8192: 122 / 119, (8, 128) 6000: 85 / 110, 8192: 139 / 137, (8, 64) 8192: 76 / 104,
// 12000: 140 / 140; not causal (28, 128) 3101: 81 / 85.  The line lies below all crossings of such lists; it looks at the shape
// only (the counts are on the device), so that the gathered and the in-place lists of the same layer take the same kernel.
// On lists of everything the other kernel is ahead from about 2.4e10 on, split / the other / the 256-row items that all
// shapes had before: (28, 128) 2048: 75 / 96 / 111, 3101: 135 / 132 / 177, 4096: 226 / 181 / 229, (28, 64) 4600: 140 / 145 /
// 186, 5900: 225 / 208 / 248, (8, 128) 7900: 197 / 210 / 226, not causal (28, 128) 2900: 209 / 192 / 209.
constexpr double kSplitWork = 6.5e10;

// Rows of a head's packed K/V buffer: whole tiles, and never a multiple of 4096 rows -- with a power-of-two
// stride between the heads, workgroups that stream different heads at the same tile index (all of them start
// at tile 0 together) hit the same cache sets and memory channels.
int fwd_npad(int rows) {
  int npad = (int)align_up(rows, kTileN);
  if (npad % 4096 == 0) npad += kTileN;
  return npad;
}

struct FwdWs {
  void* Kp;
  void* Vp;
  int* sched;
  int* qvis;
};

FwdWs carve_fwd(Arena& a, const Layer& L, int dtype, int heads, int npad, bool sparse) {
  FwdWs w;
  const size_t es = dtype == OMNI_BF16 ? 2 : 4;
  const size_t rows = (size_t)L.B * heads * npad;
  w.Kp = a.take<unsigned char>(rows * L.D * es);
  w.Vp = a.take<unsigned char>(rows * L.D * es);
  w.sched = a.take<int>(sched_ints(L.B * L.Hq, L.N, dtype == OMNI_BF16 ? kFastTileM : kTileM));
  w.qvis = sparse ? a.take<int>((size_t)L.B * L.Hq * L.N) : nullptr;
  return w;
}

unsigned split_grid(const Layer& L) { return (unsigned)(L.B * L.Hq) * (unsigned)cdiv(L.N, kSplitRows); }

template <int D, bool TILEMAP>
int launch_split(const FwdParams& p, hipStream_t st) {
  ProfScope prof__(kProfAttnFwd, st);
  hipLaunchKernelGGL((attn_fwd_split_kernel<D, TILEMAP>), dim3(split_grid(p.L)), dim3(kSplitThreads),
                     0, st, p);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

// What the forward needs to know about every token: visible counts, cleared rows, the items of the work list.
Bounds fwd_bounds(const int* q_idx, const int* q_cnt, const int* klist, int klist_stride, const int* budget, int b_cap, int* qvis,
                  void* O, int elem_bytes, float* lse, int tile_m, int* sched) {
  Bounds b{};
  b.q_idx = q_idx;
  b.q_cnt = q_cnt;
  b.klist = klist;
  b.klist_stride = klist_stride;
  b.budget = budget;
  b.b_cap = b_cap;
  b.qvis = qvis;
  b.X = O;
  b.elem_bytes = elem_bytes;
  b.lse = lse;
  b.tile_m = tile_m;
  b.sched = sched;
  return b;
}

// Bounds, packs and order of the work list.  Short sequences have no list: one launch, where each of the two passes alone takes
// little longer than an empty one.  On long ones the bounds go first, so that the order, a few serial workgroups, hides under the packs.
int prepare_fwd(const Layer& L, int dtype, const PackKv& kv, const Bounds& bn, bool split, int queues, hipStream_t st) {
  if (split) return run_prepare(L, dtype, false, &kv, nullptr, &bn, nullptr, nullptr, st);
  const int rc = run_prepare(L, dtype, false, nullptr, nullptr, &bn, nullptr, nullptr, st);
  if (rc != OMNI_OK) return rc;
  const Order order = make_order(L, bn.q_cnt, bn.tile_m, bn.sched, queues);
  return run_prepare(L, dtype, false, &kv, nullptr, nullptr, &order, nullptr, st);
}

template <typename T, int D>
int launch_fwd(const Layer& L, const void* Q, const void* K, const void* V, const int* q_idx, const int* q_cnt,
               const int* kv_idx, const int* budget, int b_cap, void* O, float* lse, void* ws, bool sparse,
               hipStream_t st) {
  Arena a(ws);
  const int heads = sparse ? L.Hq : L.Hkv;
  const int npad = fwd_npad(sparse ? b_cap : L.N);
  FwdWs w = carve_fwd(a, L, sizeof(T) == 2 ? OMNI_BF16 : OMNI_F32, heads, npad, sparse);
  // short sequences: 32-row items without a work list
  const bool split = sizeof(T) == 2 ? sparse && short_route(attention_work(L) <= kSplitWork) : f32_short(L);
  FwdParams p;
  p.Q = Q;
  p.O = O;
  p.lse = lse;
  p.L = L;
  p.q_idx = q_idx;
  p.q_cnt = q_cnt;
  p.Kp = w.Kp;
  p.Vp = w.Vp;
  p.budget = budget;
  p.b_cap = b_cap;
  p.npad = npad;
  p.per_q_head = sparse ? 1 : 0;
  p.identity_keys = sparse ? 0 : 1;
  p.sched = w.sched;
  p.qvis = w.qvis;
  p.tile_map = nullptr;
  p.tile_stride = 0;
  constexpr bool kFast = sizeof(T) == 2;
  constexpr int tile_m = kFast ? kFastTileM : kTileM;
  p.order_off = sched_order_off(L.B * L.Hq, L.N, tile_m);
  int rc = check_work_list(L, tile_m);
  if (rc != OMNI_OK) return rc;
  {
    constexpr int dt = kFast ? OMNI_BF16 : OMNI_F32;
    const bool v_rows = !kFast && !split;            // V k-packed (bf16: converted to f16); for fp32 on long sequences as it is
    PackKv kv{};
    kv.K = K;
    kv.V = V;
    kv.per_q_head = sparse ? 1 : 0;
    kv.src_idx = kv_idx;
    kv.idx_stride = b_cap;
    kv.budget = budget;
    kv.b_cap = b_cap;
    kv.npad = npad;
    kv.pad_to = kTileN;
    kv.Kn = w.Kp;
    kv.Vn = v_rows ? w.Vp : nullptr;
    kv.Vt = v_rows ? nullptr : w.Vp;
    kv.k_frag = split;
    // Per-head gathered K/V: one queue per XCD, so that the workgroups on a head share its tiles in that XCD's L2
    // (16.2 -> 5.3 GB from beyond L2 per launch at 64k).  The dense baseline and the in-place
    // block lists read one copy per KV group, which the heads of a group already share: splitting them over queues only
    // costs (25.7 -> 25.9 ms dense).
    if (sparse)
      rc = prepare_fwd(L, dt, kv, fwd_bounds(q_idx, q_cnt, kv_idx, b_cap, budget, b_cap, w.qvis, O, sizeof(T), lse, tile_m,
                                             split ? nullptr : w.sched), split, kFast ? kSchedQueues : 1, st);
    else
      rc = run_prepare(L, dt, false, &kv, nullptr, nullptr, nullptr, nullptr, st);
    if (rc != OMNI_OK) return rc;
  }
  if (split) {
    if constexpr (kFast) return launch_split<D, false>(p, st);
    ProfScope prof__(kProfAttnFwd, st);
    if constexpr (!kFast) hipLaunchKernelGGL((attn_fwd_f32_kernel<D>), dim3(split_grid(L)), dim3(kSplitThreads), 0, st, p);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
  }
  if (!sparse) {
    rc = run_schedule(L, q_cnt, budget, b_cap, tile_m, w.sched, st);
    if (rc != OMNI_OK) return rc;
  }
  ProfScope prof__(kProfAttnFwd, st);
  if constexpr (kFast)
    hipLaunchKernelGGL((attn_fwd_bf16_kernel<D, false>), dim3(persistent_grid() / 2), dim3(kFastThreads), 0, st, p);
  else
    hipLaunchKernelGGL((attn_fwd_f32_long_kernel<D>), dim3(persistent_grid()), dim3(kThreads), 0, st, p);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

// ---- in-place variant for block lists (the paper's block-sparse kernel: no gather)

struct BlockFwdWs {
  FwdWs f;
  int* klist;       // [B*Hq, blk_cap * block] token index of every entry of the heads' key lists
  int* vbudget;     // [B] their length
  int* tile_map;    // [B*Hq, blk_cap * block / 64]
};

BlockFwdWs carve_block_fwd(Arena& a, const Layer& L, int cap_keys) {
  BlockFwdWs w;
  w.f = carve_fwd(a, L, OMNI_BF16, L.Hkv, fwd_npad(L.N), false);
  const size_t BH = (size_t)L.B * L.Hq;
  w.f.qvis = a.take<int>(BH * L.N);
  w.klist = a.take<int>(BH * cap_keys);
  w.vbudget = a.take<int>(L.B);
  w.tile_map = a.take<int>(BH * (cap_keys / kTileN));
  return w;
}

template <int D>
int launch_fwd_blocks(const Layer& L, const void* Q, const void* K, const void* V, const int* q_idx, const int* q_cnt,
                      const int* blk_idx, const int* blk_budget, int blk_cap, int block, void* O, float* lse, void* ws,
                      hipStream_t st) {
  typedef u16 T;
  Arena a(ws);
  const int tpb = block / kTileN, cap_keys = blk_cap * block;
  BlockFwdWs w = carve_block_fwd(a, L, cap_keys);
  const int npad = fwd_npad(L.N);
  // K and V of every KV head once, in the kernel's tile layouts, in token order: shared by the heads of a group
  const bool split = short_route(attention_work(L) <= kSplitWork);
  // token lists of the selected blocks (for the causal bounds) and the tile map
  int rc = run_expand_blocks(L, blk_idx, blk_budget, blk_cap, block, w.klist, w.vbudget, cap_keys, st, w.tile_map, npad / kTileN - 1);
  if (rc != OMNI_OK) return rc;
  PackKv kv{};
  kv.K = K;
  kv.V = V;
  kv.b_cap = L.N;
  kv.npad = npad;
  kv.pad_to = kTileN;
  kv.Kn = w.f.Kp;
  kv.Vt = w.f.Vp;
  rc = prepare_fwd(L, OMNI_BF16, kv, fwd_bounds(q_idx, q_cnt, w.klist, cap_keys, w.vbudget, cap_keys, w.f.qvis, O, sizeof(T), lse,
                                                kFastTileM, split ? nullptr : w.f.sched), split, 1, st);
  if (rc != OMNI_OK) return rc;
  FwdParams p;
  p.Q = Q;
  p.O = O;
  p.lse = lse;
  p.L = L;
  p.q_idx = q_idx;
  p.q_cnt = q_cnt;
  p.Kp = w.f.Kp;
  p.Vp = w.f.Vp;
  p.budget = w.vbudget;
  p.b_cap = cap_keys;
  p.npad = npad;
  p.per_q_head = 0;
  p.identity_keys = 0;
  p.sched = w.f.sched;
  p.qvis = w.f.qvis;
  p.tile_map = w.tile_map;
  p.tile_stride = blk_cap * tpb;
  p.order_off = sched_order_off(L.B * L.Hq, L.N, kFastTileM);
  if (split) return launch_split<D, true>(p, st);
  {
    ProfScope prof__(kProfAttnFwd, st);
    hipLaunchKernelGGL((attn_fwd_bf16_kernel<D, true>), dim3(persistent_grid() / 2), dim3(kFastThreads), 0, st, p);
    OMNI_LAUNCH_CHECK();
  }
  return OMNI_OK;
}

}  // namespace

size_t attn_fwd_blocks_ws(const Layer& L, int cap_keys) {
  Arena a(nullptr);
  carve_block_fwd(a, L, cap_keys);
  return a.used();
}

int attn_fwd_blocks_max_keys() { return kMaxMapTiles * kTileN; }

int run_attn_fwd_blocks(const Layer& L, const void* Q, const void* K, const void* V, const int* q_idx, const int* q_cnt,
                        const int* blk_idx, const int* blk_budget, int blk_cap, int block, void* O, float* lse,
                        void* ws, hipStream_t st) {
  if (L.D == 128)
    return launch_fwd_blocks<128>(L, Q, K, V, q_idx, q_cnt, blk_idx, blk_budget, blk_cap, block, O, lse, ws, st);
  return launch_fwd_blocks<64>(L, Q, K, V, q_idx, q_cnt, blk_idx, blk_budget, blk_cap, block, O, lse, ws, st);
}

size_t attn_fwd_ws(const Layer& L, int dtype, int b_cap, bool sparse) {
  Arena a(nullptr);
  carve_fwd(a, L, dtype, sparse ? L.Hq : L.Hkv, fwd_npad(sparse ? b_cap : L.N), sparse);
  return a.used();
}

int run_attn_fwd(const Layer& L, int dtype, const void* Q, const void* K, const void* V, const int* q_idx,
                 const int* q_cnt, const int* kv_idx, const int* budget, int b_cap, void* O, float* lse, void* ws,
                 bool sparse, hipStream_t st) {
  if (dtype == OMNI_BF16) {
    if (L.D == 128)
      return launch_fwd<u16, 128>(L, Q, K, V, q_idx, q_cnt, kv_idx, budget, b_cap, O, lse, ws, sparse, st);
    return launch_fwd<u16, 64>(L, Q, K, V, q_idx, q_cnt, kv_idx, budget, b_cap, O, lse, ws, sparse, st);
  }
  if (L.D == 128)
    return launch_fwd<float, 128>(L, Q, K, V, q_idx, q_cnt, kv_idx, budget, b_cap, O, lse, ws, sparse, st);
  return launch_fwd<float, 64>(L, Q, K, V, q_idx, q_cnt, kv_idx, budget, b_cap, O, lse, ws, sparse, st);
}

}  // namespace omni
