// Builds the cost-sorted work list described in sched.h, and the visibility bounds it is priced by: two small kernels, no
// host sync.
#include "sched.h"

#include <algorithm>

namespace omni {

namespace {

constexpr int kThreads = 256;

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

// grid: (cdiv(max(N, npad), 256), B*Hq, 1 to 3).  z = 1: a wavefront owns 64 tokens and sets those of its rows that the window
// of the kept-query list does not show to zero (one that it misses is set to zero too, and written again by the attention).
// z = 0 and 2: a wavefront owns 64 kept queries, or 64 slots of the key list, and finds by search what each one sees.  Every
// entry of qvis and kfirst up to the counts, and every work item, is written from its own position, so that a list that
// repeats an index or (without the causal mask, where nothing has to be searched) is in any order gives what it means, and
// no list leaves an entry unwritten that a kernel then takes for a size.  Bound by the stores of the zeros (375 MB in all at
// 64k, three quarters of the rows dropped: 5.5 TB/s); the searches of the other wavefronts hide under them.  It took the
// place of a search kernel, a clearing pass over all rows, the pricing of the items and, in the backward, a fill and a
// scatter of the slot map: 28 heads, d = 128, 64k forward 88 -> 67 us, 32k forward and backward 111 -> 65 us; d = 64, two
// clips of 3101, forward and backward 43 -> 14 us.
__global__ __launch_bounds__(kThreads) void bounds_kernel(Layer L, Bounds p) {
  const int bh = blockIdx.y, b = bh / L.Hq, i = bh % L.Hq, lane = lane_id();
  const int r0 = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kThreads + (threadIdx.x & ~63))), n = r0 + lane;
  const int nq = p.q_cnt[bh];
  const int* qlist = p.q_idx + (long long)bh * L.N;
  if (blockIdx.z == 1) {
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
  if (blockIdx.z == 2) {                           // slots: who is the first to see the key (pads: nobody)
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

// grid: B*Hq.  The items of a head with costs estimated from their position (no key lists: the dense baseline).
__global__ __launch_bounds__(64) void sched_estimate_kernel(const int* __restrict__ q_cnt, const int* __restrict__ budget,
                                                            int b_cap, Layer L, int tile_m, int* __restrict__ sched) {
  const int bh = blockIdx.x;
  const int nt = tiles_of(q_cnt, bh, L.N, tile_m), before = items_before(q_cnt, bh, L.N, tile_m);
  int nk = budget ? budget[budget_slot(L.bph, bh / L.Hq, bh)] : L.N;
  nk = nk < 0 ? 0 : (nk > b_cap ? b_cap : nk);
  int2* items = reinterpret_cast<int2*>(sched + kSchedItems);
  for (int tq = threadIdx.x; tq < nt; tq += 64)
    items[before + tq] = make_int2((int)(((unsigned)bh << 16) | (unsigned)tq), sched_estimate(tq, nt, nk, L.causal));
}

// grid: cdiv(cap, kRankItems).  The hand-out order of the items: an item's rank among the keys (all distinct) is its
// place.  Every workgroup places the heads on the queues for itself (a few hundred instructions: less than a launch),
// the first one writes the header.  One launch where there were three (prefix, placement, rank): 31 -> 18 us at 64k, 29 -> 11 at 32k.
constexpr int kRankLanes = 16;
constexpr int kRankItems = kThreads / kRankLanes;           // items per workgroup
struct QueuePlaces {
  int place[kSchedMaxQueuedHeads], cost[kSchedMaxQueuedHeads], items[kSchedMaxQueuedHeads], order[kSchedMaxQueuedHeads];
};
__global__ __launch_bounds__(kThreads) void sched_order_kernel(const int* __restrict__ q_cnt, int BH, int N, int tile_m,
                                                               int queues, int workgroups, size_t order_off,
                                                               int* __restrict__ sched) {
  constexpr int kTile = 2048;                               // keys staged per pass: a 64k layer's list in one
  __shared__ unsigned long long tile[kTile];
  __shared__ QueuePlaces sh;
  __shared__ int s_wave[kThreads / 64], s_big[kThreads / 64], s_head[kThreads / 64];
  __shared__ long long s_tot[kThreads / 64];
  __shared__ int s_end[kSchedQueues];
  const int2* items = reinterpret_cast<const int2*>(sched + kSchedItems);
  const int wave = threadIdx.x >> 6;
  // number of items
  int n = 0;
  for (int bh = threadIdx.x; bh < BH; bh += kThreads) n += tiles_of(q_cnt, bh, N, tile_m);
  n = wave_sum(n);
  if (lane_id() == 0) s_wave[wave] = n;
  __syncthreads();
  n = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) n += s_wave[w];
  if (blockIdx.x > 0 && (int)blockIdx.x * kRankItems >= n) return;
  bool queued = queues > 1 && BH <= kSchedMaxQueuedHeads, by_head = true;
  if (queued) {
    // head costs; whether queues pay
    for (int bh = threadIdx.x; bh < BH; bh += kThreads) {
      sh.cost[bh] = 0;
      sh.items[bh] = tiles_of(q_cnt, bh, N, tile_m);
    }
    __syncthreads();
    int big = 0;
    long long tot = 0;
    constexpr int kBatch = 4;                               // loads in flight
    for (int j0 = 0; j0 < n; j0 += kBatch * kThreads) {
      int2 it[kBatch];
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const int j = j0 + e * kThreads + (int)threadIdx.x;
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
    for (int bh = threadIdx.x; bh < BH; bh += kThreads) head = max(head, sh.cost[bh]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      big = max(big, __shfl_xor(big, o, 64));
      head = max(head, __shfl_xor(head, o, 64));
      tot += __shfl_xor(tot, o, 64);
    }
    if (lane_id() == 0) {
      s_big[wave] = big;
      s_head[wave] = head;
      s_tot[wave] = tot;
    }
    __syncthreads();
    big = head = 0;
    tot = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
      big = max(big, s_big[w]);
      head = max(head, s_head[w]);
      tot += s_tot[w];
    }
    queued = sched_queues_pay(tot, head, queues);
    by_head = sched_long_enough(tot, big, workgroups);
    if (queued) {
      const int shift = sched_cost_shift(tot);
      for (int bh = threadIdx.x; bh < BH; bh += kThreads) {     // rank of a head: cost descending, index ascending
        const int mine = sh.cost[bh];
        int r = 0;
        for (int j = 0; j < BH; ++j) r += (sh.cost[j] > mine || (sh.cost[j] == mine && j < bh)) ? 1 : 0;
        sh.order[r] = bh;
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
          const int ni = sh.items[bh];
#pragma unroll
          for (int r = 0; r < kSchedQueues; ++r)               // compile-time indices keep the arrays in registers
            if (r == q) {
              sh.place[bh] = (r << 16) | heads[r];
              heads[r] += 1;
              load[r] += c;
              count[r] += ni;
            }
        }
        int start = 0;
#pragma unroll
        for (int q = 0; q < kSchedQueues; ++q) s_end[q] = start += count[q];
      }
      __syncthreads();
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < kSchedQueues) {
    const int q = threadIdx.x;
    sched[kSchedEnd + q] = queued ? s_end[q] : n;
    sched[kSchedCursor + q] = q == 0 ? 0 : (queued ? s_end[q - 1] : n);
    if (q == 0) sched[kSchedTotal] = n;
  }
  auto key_of = [&](int2 it, int id) {
    const unsigned place = queued ? (unsigned)sh.place[(unsigned)it.x >> 16] : 0u;
    return sched_key(it.y, id, by_head ? place : place & 0xffff0000u);
  };
  const int id = blockIdx.x * kRankItems + threadIdx.x / kRankLanes, sub = threadIdx.x % kRankLanes;
  const int2 own = id < n ? items[id] : make_int2(0, 0);
  const unsigned long long mine = key_of(own, id);
  int rank = 0;
  for (int j0 = 0; j0 < n; j0 += kTile) {                   // uniform trip count: every thread helps to stage
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kTile / kThreads; ++u) {            // independent loads: one memory latency per pass
      const int j = j0 + u * kThreads + (int)threadIdx.x;
      tile[u * kThreads + threadIdx.x] = j < n ? key_of(items[j], j) : 0ull;
    }
    __syncthreads();
    const int m = min(kTile, n - j0);
#pragma unroll 16
    for (int j = sub; j < m; j += kRankLanes) rank += tile[j] > mine ? 1 : 0;     // unrolled: LDS reads in flight together
  }
#pragma unroll
  for (int o = 1; o < kRankLanes; o <<= 1) rank += __shfl_xor(rank, o, 64);
  if (id < n && sub == 0) sched[order_off + rank] = own.x;
}

}  // namespace

int check_work_list(const Layer& L, int tile_m) {
  if (L.B * L.Hq >= 65536 || cdiv(L.N, tile_m) >= 65536) OMNI_FAIL(OMNI_ERR_UNSUPPORTED, "work list: too many heads or tiles");
  return OMNI_OK;
}

int run_bounds(const Layer& L, const Bounds& p, hipStream_t st) {
  const int BH = L.B * L.Hq, n = p.kfirst ? max(L.N, p.npad) : L.N;
  hipLaunchKernelGGL(bounds_kernel, dim3(cdiv(n, kThreads), BH, p.kfirst ? 3 : p.X ? 2 : 1), dim3(kThreads), 0, st, L, p);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

int run_order(const Layer& L, const int* q_cnt, int tile_m, int* sched, hipStream_t st, int queues) {
  const int BH = L.B * L.Hq;
  const size_t cap = sched_cap(BH, L.N, tile_m);
  hipLaunchKernelGGL(sched_order_kernel, dim3((unsigned)cdiv(cap, (size_t)kRankItems)), dim3(kThreads), 0, st, q_cnt, BH,
                     L.N, tile_m, queues, persistent_grid() / 2, sched_order_off(BH, L.N, tile_m), sched);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

int run_schedule(const Layer& L, const int* q_cnt, const int* budget, int b_cap, int tile_m, int* sched, hipStream_t st) {
  const int BH = L.B * L.Hq;
  hipLaunchKernelGGL(sched_estimate_kernel, dim3(BH), dim3(64), 0, st, q_cnt, budget, b_cap, L, tile_m, sched);
  OMNI_LAUNCH_CHECK();
  return run_order(L, q_cnt, tile_m, sched, st);
}

HostWorkList sched_build_host(const int* q_cnt, const int* budget, int B, int Hq, int N, int b_cap, int causal, int tile_m,
                              int queues, int workgroups) {
  const int BH = B * Hq;
  std::vector<int> packed, costs, head_items(BH);
  std::vector<long long> head_cost(BH);
  long long total = 0, largest_head = 0, largest_item = 0;
  for (int bh = 0; bh < BH; ++bh) {
    const int nq = q_cnt ? q_cnt[bh] : N, nt = nq > 0 ? (nq + tile_m - 1) / tile_m : 0;
    int nk = budget ? budget[bh / Hq] : N;
    nk = nk < 0 ? 0 : (nk > b_cap ? b_cap : nk);
    for (int tq = 0; tq < nt; ++tq) {
      packed.push_back((int)(((unsigned)bh << 16) | (unsigned)tq));
      costs.push_back(sched_estimate(tq, nt, nk, causal));
      head_cost[bh] += costs.back();
      largest_item = std::max(largest_item, (long long)costs.back());
    }
    head_items[bh] = nt;
    total += head_cost[bh];
    largest_head = std::max(largest_head, head_cost[bh]);
  }
  const int items = (int)packed.size();
  const bool queued = queues > 1 && BH <= kSchedMaxQueuedHeads && sched_queues_pay(total, largest_head, queues);
  const bool by_head = sched_long_enough(total, largest_item, workgroups);
  std::vector<unsigned> place(BH, 0u);
  int count[kSchedQueues] = {};
  if (queued) {
    std::vector<int> heads(BH);                          // by cost, lower index first among equals
    for (int bh = 0; bh < BH; ++bh) heads[bh] = bh;
    std::stable_sort(heads.begin(), heads.end(), [&](int x, int y) { return head_cost[x] > head_cost[y]; });
    const int shift = sched_cost_shift(total);
    unsigned load[kSchedQueues];
    int placed[kSchedQueues] = {};
    for (int q = 0; q < kSchedQueues; ++q) load[q] = q < queues ? (unsigned)q : 0xffffffffu;
    for (int bh : heads) {
      const int q = (int)(*std::min_element(load, load + kSchedQueues) & 7u);
      place[bh] = ((unsigned)q << 16) | (unsigned)placed[q]++;
      load[q] += (unsigned)(head_cost[bh] >> shift) << 3;
      count[q] += head_items[bh];
    }
  } else {
    count[0] = items;
  }
  HostWorkList list;
  for (int q = 0, end = 0; q < kSchedQueues; ++q) list.end[q] = end += count[q];
  std::vector<int> idx(items);
  for (int i = 0; i < items; ++i) idx[i] = i;
  auto key = [&](int id) {
    const unsigned at = place[(unsigned)packed[id] >> 16];
    return sched_key(costs[id], id, by_head ? at : at & 0xffff0000u);
  };
  std::sort(idx.begin(), idx.end(), [&](int x, int y) { return key(x) > key(y); });
  for (int id : idx) {
    list.packed.push_back(packed[id]);
    list.cost.push_back(costs[id]);
  }
  return list;
}

int persistent_grid() {
  static int grid = 0;
  if (grid == 0) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    grid = 2 * cus;
  }
  return grid;
}

}  // namespace omni
