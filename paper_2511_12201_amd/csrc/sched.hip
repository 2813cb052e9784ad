// The cost-sorted work list described in sched.h where no pack precedes its order (the dense baseline), and the same list on
// the host.
#include "sched_dev.h"

#include <algorithm>

namespace omni {

namespace {

constexpr int kThreads = 256;

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

// grid: cdiv(cap, kThreads / kRankLanes)
__global__ __launch_bounds__(kThreads) void sched_order_kernel(Order od) {
  __shared__ OrderShared<kThreads> sh;
  order_block<kThreads>(od, blockIdx.x, sh);
}

}  // namespace

int check_work_list(const Layer& L, int tile_m) {
  if (L.B * L.Hq >= 65536 || cdiv(L.N, tile_m) >= 65536) OMNI_FAIL(OMNI_ERR_UNSUPPORTED, "work list: too many heads or tiles");
  return OMNI_OK;
}

Order make_order(const Layer& L, const int* q_cnt, int tile_m, int* sched, int queues) {
  Order od;
  od.q_cnt = q_cnt;
  od.BH = L.B * L.Hq;
  od.N = L.N;
  od.tile_m = tile_m;
  od.queues = queues;
  od.workgroups = persistent_grid() / 2;
  od.order_off = sched_order_off(od.BH, L.N, tile_m);
  od.sched = sched;
  return od;
}

int run_schedule(const Layer& L, const int* q_cnt, const int* budget, int b_cap, int tile_m, int* sched, hipStream_t st) {
  const int BH = L.B * L.Hq;
  hipLaunchKernelGGL(sched_estimate_kernel, dim3(BH), dim3(64), 0, st, q_cnt, budget, b_cap, L, tile_m, sched);
  OMNI_LAUNCH_CHECK();
  hipLaunchKernelGGL(sched_order_kernel, dim3((unsigned)cdiv(sched_cap(BH, L.N, tile_m), (size_t)(kThreads / kRankLanes))),
                     dim3(kThreads), 0, st, make_order(L, q_cnt, tile_m, sched));
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
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
