// Device code of the work lists (sched.h): what every position sees, the order of the items, the key kernel's list.  Blocks of
// a launch that also holds the packs (pack.hip) or, for the dense baseline, of a kernel of its own (sched.hip).
#pragma once

#include "sched.h"

namespace omni {

namespace {

__device__ __forceinline__ int tiles_of(const int* __restrict__ q_cnt, int bh, int N, int tile_m) {
  const int nq = q_cnt ? q_cnt[bh] : N;
  return nq > 0 ? (nq + tile_m - 1) / tile_m : 0;
}

// Items of the heads before bh; every lane of the wavefront gets the sum.
__device__ __forceinline__ int items_before(const int* __restrict__ q_cnt, int bh, int N, int tile_m) {
  int s = 0;
  for (int i = lane_id(); i < bh; i += 64) s += tiles_of(q_cnt, i, N, tile_m);
  return __builtin_amdgcn_readlane((int)wave_scan((unsigned)s), 63);
}

// First position of the ascending a[0, n) with a[pos] >= v, by a whole wavefront: 64 probes a step.
__device__ __forceinline__ int wave_lower_bound(const int* __restrict__ a, int n, int v) {
  int lo = 0, hi = n;
  while (hi - lo > 64) {
    const int step = (hi - lo + 63) >> 6, at = lo + (lane_id() + 1) * step - 1;
    const int below = (int)__popcll(__ballot(at < hi && a[at] < v));
    lo += below * step;
    hi = min(lo + step, hi);
  }
  const int at = lo + lane_id();
  return lo + (int)__popcll(__ballot(at < hi && a[at] < v));
}

__device__ __forceinline__ unsigned wave_or(unsigned v) {
  v |= dpp_or_zero<0x111, 0xf>(v);
  v |= dpp_or_zero<0x112, 0xf>(v);
  v |= dpp_or_zero<0x114, 0xf>(v);
  v |= dpp_or_zero<0x118, 0xf>(v);
  v |= dpp_or_zero<0x142, 0xa>(v);
  v |= dpp_or_zero<0x143, 0xc>(v);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// Which of the tokens [r0, r0 + 64) the list holds, one bit each.  A set bit is always an entry; of a list that is not
// strictly ascending some entries may be missed.
__device__ __forceinline__ unsigned long long list_window(const int* __restrict__ list, int n, int r0) {
  const int at = wave_lower_bound(list, n, r0) + lane_id();
  const unsigned o = at < n ? (unsigned)(list[at] - r0) : 64u;
  const unsigned lo = wave_or(o < 32u ? 1u << o : 0u), hi = wave_or(o >= 32u && o < 64u ? 1u << (o & 31u) : 0u);
  return ((unsigned long long)hi << 32) | lo;
}

// Per lane: first position of the ascending a[0, n) with a[pos] >= v, for values that ascend from lane to lane: the wavefront
// finds where its first and its last value fall, a lane searches between.  Whatever the list holds the result is in [0, n].
__device__ __forceinline__ int lanes_lower_bound(const int* __restrict__ a, int n, int v) {
  int lo = wave_lower_bound(a, n, __builtin_amdgcn_readfirstlane(v));
  int hi = max(lo, wave_lower_bound(a, n, __builtin_amdgcn_readlane(v, 63)));
  while (__any(lo < hi)) {
    const int mid = (lo + hi) >> 1;
    if (lo < hi) {
      if (a[mid] < v) lo = mid + 1;
      else hi = mid;
    }
  }
  return lo;
}

// Block (bx, bh, role) of cdiv(max(N, npad), NT) x B*Hq x 1 to 3 blocks.  Role 1: a wavefront owns 64 tokens and sets those of its rows that the window
// of the kept-query list does not show to zero (one that it misses is set to zero too, and written again by the attention).
// Roles 0 and 2: a wavefront owns 64 kept queries, or 64 slots of the key list, and finds by search what each one sees.  Every
// entry of qvis and kfirst up to the counts, and every work item, is written from its own position, so that a list that
// repeats an index or (without the causal mask, where nothing has to be searched) is in any order gives what it means, and
// no list leaves an entry unwritten that a kernel then takes for a size.  Bound by the stores of the zeros (375 MB in all at
// 64k, three quarters of the rows dropped: 5.5 TB/s); the searches of the other wavefronts hide under them.  It took the
// place of a search kernel, a clearing pass over all rows, the pricing of the items and, in the backward, a fill and a
// scatter of the slot map: 28 heads, d = 128, 64k forward 88 -> 67 us, 32k forward and backward 111 -> 65 us; d = 64, two
// clips of 3101, forward and backward 43 -> 14 us.
template <int NT>
__device__ __forceinline__ void bounds_block(const Layer& L, const Bounds& p, int bx, int bh, int role) {
  const int b = bh / L.Hq, i = bh % L.Hq, lane = lane_id();
  const int r0 = __builtin_amdgcn_readfirstlane((int)(bx * NT + (threadIdx.x & ~63))), n = r0 + lane;
  const int nq = p.q_cnt[bh];
  const int* qlist = p.q_idx + (long long)bh * L.N;
  if (role == 1) {
    if (r0 >= L.N) return;
    const unsigned long long kept = list_window(qlist, nq, r0);
    const int per_row = L.D * p.elem_bytes / 16;   // lanes that store one row: 8, 16 or 32
    char* base = static_cast<char*>(p.X) + (b * L.qs[0] + i * L.qs[1]) * p.elem_bytes + lane % per_row * 16;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int r = lane / per_row; r < 64; r += 64 / per_row)
      if (r0 + r < L.N && !(kept >> r & 1)) *reinterpret_cast<u32x4*>(base + (r0 + r) * L.qs[2] * p.elem_bytes) = zero;
    if (p.lse && n < L.N && !(kept >> lane & 1)) p.lse[(long long)bh * L.N + n] = -INFINITY;
    return;
  }
  const int nkeys = max(min(p.budget[budget_slot(L.bph, b, bh)], p.b_cap), 0);
  const int* klist = p.klist + (long long)bh * p.klist_stride;
  if (role == 2) {                           // slots: who is the first to see the key (pads: nobody)
    if (r0 >= p.npad) return;
    const int tok = r0 < nkeys ? klist[min(n, nkeys - 1)] : 0;
    const int first = r0 < nkeys && L.causal ? lanes_lower_bound(qlist, nq, tok) : 0;
    if (n < p.npad) p.kfirst[(long long)bh * p.npad + n] = n < nkeys ? first : nq;
    if (n < nkeys && (unsigned)tok < (unsigned)L.N) p.inv[(long long)bh * L.N + tok] = n;
    return;
  }
  if (r0 >= nq) return;
  const int row = qlist[min(n, nq - 1)];           // kept queries: how many keys they see
  const int visible = L.causal ? lanes_lower_bound(klist, nkeys, row + 1) : nkeys;
  if (p.qvis && n < nq) p.qvis[(long long)bh * L.N + n] = visible;
  const bool last = n < nq && (n % p.tile_m == p.tile_m - 1 || n == nq - 1);       // last row of a work item
  if (!p.sched || !__any(last)) return;
  const int before = items_before(p.q_cnt, bh, L.N, p.tile_m);
  if (last) {
    const int tq = n / p.tile_m;
    reinterpret_cast<int2*>(p.sched + kSchedItems)[before + tq] =
        make_int2((int)(((unsigned)bh << 16) | (unsigned)tq), (visible + kTileN - 1) / kTileN);
  }
}

// Block bx of cdiv(cap, NT / kRankLanes) blocks.  The hand-out order of the items: an item's rank among the keys (all distinct) is its
// place.  Every workgroup places the heads on the queues for itself (a few hundred instructions: less than a launch),
// the first one writes the header.  One launch where there were three (prefix, placement, rank): 31 -> 18 us at 64k, 29 -> 11 at 32k.
// The serial placement takes a head's number of items from LDS: as a load for each head it was 56 us for 224 heads and 80 beside
// the packs, which it then did not hide under.  Forward call, 28 heads a sequence, d = 128, before / now in us: 8 sequences of
// 3000 334 / 280, 32 of 2000 982 / 800, one of 16384 420 / 413.
constexpr int kRankLanes = 16;
constexpr int kRankTile = 1024;                             // keys staged per pass
// 16.5 KB with 256 threads, 16.6 with 384 or 512.  The packs of the same launches need 16.6 KB (bf16, d = 128; 33 where Q and dO
// are packed too), 8.4 KB (bf16 forward, d = 64) or 256 bytes (fp32); the wavefronts of eight workgroups of 256 threads fill a CU
// in any case, with 133 of its 160 KB.
template <int NT>
struct OrderShared {
  unsigned long long tile[kRankTile];
  int cost[kSchedMaxQueuedHeads];
  u16 place[kSchedMaxQueuedHeads], order[kSchedMaxQueuedHeads];        // place = queue << 13 | position in it
  long long tot[NT / 64];
  int wave[NT / 64], big[NT / 64], head[NT / 64], end[kSchedQueues];
};
template <int NT>
__device__ __forceinline__ void order_block(const Order& od, int bx, OrderShared<NT>& sh) {
  constexpr int kRankItems = NT / kRankLanes;               // items per workgroup
  const int* __restrict__ q_cnt = od.q_cnt;
  int* __restrict__ sched = od.sched;
  const int BH = od.BH, N = od.N, tile_m = od.tile_m, queues = od.queues;
  const int2* items = reinterpret_cast<const int2*>(sched + kSchedItems);
  const int wave = threadIdx.x >> 6;
  // number of items
  int n = 0;
  for (int bh = threadIdx.x; bh < BH; bh += NT) n += tiles_of(q_cnt, bh, N, tile_m);
  n = wave_sum(n);
  if (lane_id() == 0) sh.wave[wave] = n;
  __syncthreads();
  n = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) n += sh.wave[w];
  if (bx > 0 && bx * kRankItems >= n) return;
  bool queued = queues > 1 && BH <= kSchedMaxQueuedHeads, by_head = true;
  if (queued) {
    // head costs; whether queues pay
    for (int bh = threadIdx.x; bh < BH; bh += NT) sh.cost[bh] = 0;
    __syncthreads();
    int big = 0;
    long long tot = 0;
    constexpr int kBatch = 4;                               // loads in flight
    for (int j0 = 0; j0 < n; j0 += kBatch * NT) {
      int2 it[kBatch];
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const int j = j0 + e * NT + (int)threadIdx.x;
        it[e] = j < n ? items[j] : make_int2(0, 0);
      }
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const int bh = (int)((unsigned)it[e].x >> 16), first = __builtin_amdgcn_readfirstlane(bh);
        big = max(big, it[e].y);
        tot += it[e].y;
        if (__all(bh == first || it[e].y == 0)) {           // 64 consecutive items belong to one head most of the time
          const int c = (int)wave_scan((unsigned)it[e].y);
          if (lane_id() == 63 && c) atomicAdd(&sh.cost[first], c);
        } else if (it[e].y) {
          atomicAdd(&sh.cost[bh], it[e].y);
        }
      }
    }
    __syncthreads();
    int head = 0;
    for (int bh = threadIdx.x; bh < BH; bh += NT) head = max(head, sh.cost[bh]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      big = max(big, __shfl_xor(big, o, 64));
      head = max(head, __shfl_xor(head, o, 64));
      tot += __shfl_xor(tot, o, 64);
    }
    if (lane_id() == 0) {
      sh.big[wave] = big;
      sh.head[wave] = head;
      sh.tot[wave] = tot;
    }
    __syncthreads();
    big = head = 0;
    tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      big = max(big, sh.big[w]);
      head = max(head, sh.head[w]);
      tot += sh.tot[w];
    }
    queued = sched_queues_pay(tot, head, queues);
    by_head = sched_long_enough(tot, big, od.workgroups);
    if (queued) {
      const int shift = sched_cost_shift(tot);
      for (int bh = threadIdx.x; bh < BH; bh += NT) {     // rank of a head: cost descending, index ascending
        const int mine = sh.cost[bh];
        int r = 0;
        for (int j = 0; j < BH; ++j) r += (sh.cost[j] > mine || (sh.cost[j] == mine && j < bh)) ? 1 : 0;
        sh.order[r] = (u16)bh;
        sh.place[bh] = (u16)tiles_of(q_cnt, bh, N, tile_m);       // until the head is placed
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        unsigned load[kSchedQueues];           // load << 3 | queue: the least loaded queue is one unsigned minimum
        int heads[kSchedQueues], count[kSchedQueues];
#pragma unroll
        for (int q = 0; q < kSchedQueues; ++q) load[q] = q < queues ? (unsigned)q : 0xffffffffu, heads[q] = 0, count[q] = 0;
        for (int k = 0; k < BH; ++k) {
          const int bh = sh.order[k];
          unsigned m = load[0];
#pragma unroll
          for (int r = 1; r < kSchedQueues; ++r) m = min(m, load[r]);
          const int q = (int)(m & 7u);
          const unsigned c = (unsigned)(sh.cost[bh] >> shift) << 3;
          const int ni = sh.place[bh];
#pragma unroll
          for (int r = 0; r < kSchedQueues; ++r)               // compile-time indices keep the arrays in registers
            if (r == q) {
              sh.place[bh] = (u16)(r << 13 | heads[r]);
              heads[r] += 1;
              load[r] += c;
              count[r] += ni;
            }
        }
        int start = 0;
#pragma unroll
        for (int q = 0; q < kSchedQueues; ++q) sh.end[q] = start += count[q];
      }
      __syncthreads();
    }
  }
  if (bx == 0 && threadIdx.x < kSchedQueues) {
    const int q = threadIdx.x;
    sched[kSchedEnd + q] = queued ? sh.end[q] : n;
    sched[kSchedCursor + q] = q == 0 ? 0 : (queued ? sh.end[q - 1] : n);
    if (q == 0) sched[kSchedTotal] = n;
  }
  auto key_of = [&](int2 it, int id) {
    const unsigned at = queued ? (unsigned)sh.place[(unsigned)it.x >> 16] : 0u, queue = at >> 13 << 16;
    return sched_key(it.y, id, by_head ? queue | (at & 0x1fffu) : queue);
  };
  const int id = bx * kRankItems + threadIdx.x / kRankLanes, sub = threadIdx.x % kRankLanes;
  const int2 own = id < n ? items[id] : make_int2(0, 0);
  const unsigned long long mine = key_of(own, id);
  int rank = 0;
  for (int j0 = 0; j0 < n; j0 += kRankTile) {                   // uniform trip count: every thread helps to stage
    __syncthreads();
#pragma unroll
    for (int u = 0; u < (kRankTile + NT - 1) / NT; ++u) {       // independent loads: one memory latency per pass
      const int at = u * NT + (int)threadIdx.x, j = j0 + at;
      if (at < kRankTile) sh.tile[at] = j < n ? key_of(items[j], j) : 0ull;
    }
    __syncthreads();
    const int m = min(kRankTile, n - j0);
#pragma unroll 16
    for (int j = sub; j < m; j += kRankLanes) rank += sh.tile[j] > mine ? 1 : 0;     // unrolled: LDS reads in flight together
  }
#pragma unroll
  for (int o = 1; o < kRankLanes; o <<= 1) rank += __shfl_xor(rank, o, 64);
  if (id < n && sub == 0) sched[od.order_off + rank] = own.x;
}

// Work items of the key kernel: (head, key tile, split), in dispatch order -- heads in groups of head_group,
// inside a group key tile by key tile (the first key tiles, seen by the most queries, first), the splits of a
// tile side by side.  Slot i of that order is a (head, key tile); most are empty (key tiles beyond a head's
// budget), so one workgroup lists the live ones with their splits, and the persistent key kernel pulls from
// the list: an empty workgroup would still wait for a whole CU's LDS.
// head and key tile of slot i, and how many query tiles see it (0: nothing to do)
__device__ __forceinline__ int key_slot(const Layer& L, const KeyList& p, int i, int& bh, int& ktile) {
  const int BH = L.B * L.Hq, nkt = p.npad / kKeyTile;
  const int per_group = p.head_group * nkt, grp = i / per_group, within = i % per_group;
  const int heads_here = min(p.head_group, BH - grp * p.head_group);
  if (heads_here <= 0) return 0;
  ktile = within / heads_here;
  bh = grp * p.head_group + within % heads_here;
  if (ktile >= nkt) return 0;
  if (ktile * kKeyTile >= min(p.budget[budget_slot(L.bph, bh / L.Hq, bh)], p.b_cap)) return 0;
  return max(1, cdiv(p.q_cnt[bh], kKeyQ) - p.kfirst[(long long)bh * p.npad + ktile * kKeyTile] / kKeyQ);
}

// One workgroup: the list, and the length of a split: a workgroup's share of all query tiles (a longer
// chain would outlast the others), between 5 and p.split_len (1072 tokens, 28 heads, d = 128, forward and backward at least 8 / 5
// tiles: 108 / 98 us; elsewhere level).  At 3k tokens, two sequences of 28 heads, the longest chain
// is head 0's 49 query tiles while a share is 9: dK' 87 -> 44 us, dV' 63 -> 34 us.
template <int NT>
__device__ __forceinline__ void key_list_block(const Layer& L, const KeyList& p, int (&wave_cnt)[NT / 64]) {
  const int n_slots = p.n_slots;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int bh, ktile, tiles = 0;
  for (int i = threadIdx.x; i < n_slots; i += NT) tiles += key_slot(L, p, i, bh, ktile);
  tiles = wave_sum(tiles);
  if (lane == 0) wave_cnt[wave] = tiles;
  __syncthreads();
  tiles = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) tiles += wave_cnt[w];
  const int split_len = min(p.split_len, max(5, cdiv(tiles, p.key_wgs)));
  int base = 0;
  for (int i0 = 0; i0 < n_slots; i0 += NT) {
    const int i = i0 + (int)threadIdx.x;
    const int seen = i < n_slots ? key_slot(L, p, i, bh, ktile) : 0;
    const int n_sp = seen ? key_tile_splits(seen, p.nsplit, split_len) : 0;
    const int incl = (int)wave_scan((unsigned)n_sp);
    __syncthreads();
    if (lane == 63) wave_cnt[wave] = incl;
    __syncthreads();
    int at = base + incl - n_sp;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      at += w < wave ? wave_cnt[w] : 0;
      base += wave_cnt[w];
    }
    if (n_sp) {
      const int* kfirst = p.kfirst + (long long)bh * p.npad + ktile * kKeyTile;
      const int nkeys = min(p.budget[budget_slot(L.bph, bh / L.Hq, bh)], p.b_cap) - ktile * kKeyTile;
      const int q_tiles = cdiv(p.q_cnt[bh], kKeyQ), first = kfirst[0] / kKeyQ, each = cdiv(q_tiles - first, n_sp);
      const int unmasked = nkeys < kKeyTile ? 0x7fffffff : kfirst[kKeyTile - 1];
      int4* items = reinterpret_cast<int4*>(p.klist + kKeyListHeader) + at;
      for (int sp = 0; sp < n_sp; ++sp)
        items[sp] = make_int4((bh << 16) | (ktile << 3) | sp, first + sp * each, min(each, q_tiles - first - sp * each), unmasked);
    }
  }
  if (threadIdx.x == 0) {
    p.klist[0] = 0;
    p.klist[1] = base;
    p.klist[2] = split_len;
    p.klist[kKeyListRows] = 0;
  }
}

}  // namespace

}  // namespace omni
