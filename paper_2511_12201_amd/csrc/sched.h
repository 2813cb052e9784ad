// Device-side work list for the query-tile kernels (attention forward, backward dQ).
//
// Work item = one tile (tile_m rows, 128 or 256) of a head's kept queries.  Under the causal mask the
// items differ in length by two orders of magnitude (a head's last tile streams every selected key, its
// first one tile), and a launch has only a few thousand of them for 256 persistent workgroups: handed out
// head by head, the long items of the last heads start late and a few workgroups finish them alone
// (measured: 17 % of the kernel time).  So the items are sorted by cost, longest first, and every
// workgroup pulls the next one from a single atomic counter -- the classic longest-processing-time
// rule, whose tail is bounded by the shortest items.  The cost of an item is the number of key tiles
// it streams: exact where there are index lists, estimated from the position of the tile for the dense baseline.
//
// The list can be cut into kSchedQueues queues, one per XCD (workgroups are dealt to the XCDs round-robin, so
// workgroup i sits on XCD i % 8): whole heads are assigned to queues, largest first onto the least loaded
// queue, and inside a queue the heads follow one another, each longest item first, or all its items longest first
// (sched_long_enough); one list after all if some head outweighs a queue's fair share (sched_queues_pay).  The 32 workgroups of an
// XCD then stream the K/V tiles of one head a few tiles apart and find them in the XCD's own L2 instead of
// each fetching its own copy; a workgroup whose queue is drained takes from the queue with the most items left.
// On the 64k forward this cuts the traffic from beyond L2 to a third and leaves the kernel time where it was: the
// kernel is not bound by that traffic, the queues just stop it from wasting memory bandwidth.
//
// Layout of the int array in device memory:
//   [0] unused   [1] number of items   [2..3] unused
//   [4 .. 11] cursor[q]: next position of queue q   [12 .. 19] end[q]   (one queue: cursor[0] = 0, end[0] = items)
//   [20 .. + 2 * cap]        items by id: (head << 16 | tile), cost
//   [.. + cap]               order[k] = (head << 16 | tile) of the k-th item to hand out
// with cap = BH * ceil(N / tile_m) the largest possible number of items.
#pragma once

#include <vector>

#include "common.h"

namespace omni {

constexpr int kSchedQueues = 8;
constexpr int kSchedTotal = 1, kSchedCursor = 4, kSchedEnd = kSchedCursor + kSchedQueues;
constexpr int kSchedItems = kSchedEnd + kSchedQueues;      // even: the items are read as pairs
constexpr int kSchedMaxQueuedHeads = 1024;       // more heads than this: one queue (the placement is a serial loop)

inline size_t sched_cap(int BH, int N, int tile_m) { return (size_t)BH * ((N + tile_m - 1) / tile_m); }
inline size_t sched_order_off(int BH, int N, int tile_m) { return (size_t)kSchedItems + 2 * sched_cap(BH, N, tile_m); }
inline size_t sched_ints(int BH, int N, int tile_m) { return sched_order_off(BH, N, tile_m) + sched_cap(BH, N, tile_m); }

// What the kept-query and key lists say about every position and token, by bounds_block (sched_dev.h); null: not wanted.
struct Bounds {
  const int *q_idx, *q_cnt;      // [B*Hq, N], [B*Hq]
  const int* klist;              // [B*Hq, klist_stride] token indices, the first min(budget, b_cap) of a head
  int klist_stride;
  const int* budget;
  int b_cap, npad;
  int* qvis;                     // [B*Hq, N] number of listed keys that kept query `pos` may see
  int* kfirst;                   // [B*Hq, npad] first kept-query position that may see listed key `slot` (needs inv and X)
  int* inv;                      // [B*Hq, N] slot of the token in the key list (listed tokens; the others are not written)
  void* X;                       // nullable (then lse is not written either): rows of the Q-shaped tensor (16-byte aligned)
                                 // that are not kept are set to zero
  int elem_bytes;
  float* lse;                    // [B*Hq, N] -inf for the rows that are not kept
  int tile_m;                    // rows per work item
  int* sched;                    // the items of the work list and their costs (not their order)
};
int check_work_list(const Layer& L, int tile_m);     // the items' fields are 16 bits wide: error if they do not fit

// The order of the work list from its items: queues = 1 (one longest-first list) or kSchedQueues (one list per XCD, whole
// heads per queue, where that pays).
struct Order {
  const int* q_cnt;              // [BH], null: N each
  int BH, N, tile_m, queues;
  int workgroups;                // one per CU
  size_t order_off;
  int* sched;
};
Order make_order(const Layer& L, const int* q_cnt, int tile_m, int* sched, int queues = 1);

// The work list of the bf16 key kernel of the backward (attn_bwd.hip): (head, key tile, split) in dispatch order.
constexpr int kKeyTile = 256;                // packed keys per workgroup
constexpr int kKeyQ = 64;                    // queries per tile, as the splits count them
constexpr int kKeyListHeader = 4;            // counter, number of items, query tiles per split, counter of the 32-row dQ items
constexpr int kKeyListRows = 3;
// An item is four ints, all that a workgroup has to know before its first load: head << 16 | key tile << 3 | split, first query
// tile, number of query tiles, first query position from which on nothing is masked.
constexpr int kKeyItemInts = 4;
struct KeyList {
  const int *q_cnt, *budget;
  int b_cap, npad;
  const int* kfirst;             // [B*Hq, npad], as in Bounds
  int head_group;                // heads per dispatch group
  int nsplit, split_len;         // most workgroups that share the query tiles of a key tile, tiles per split at most
  int key_wgs;                   // workgroups that share the items
  int n_slots;
  int* klist;
};
// A key tile seen by many query tiles (the first tiles of a head that keeps every query: 512 query tiles at 32k,
// against a few dozen for most workgroups) is shared by several workgroups, each with a contiguous range of the
// query tiles and a partial-gradient plane of its own; the group reduction adds the planes in split order.
__host__ __device__ inline int key_tile_splits(int n_qtiles, int max_splits, int split_len) {
  const int s = n_qtiles / split_len;
  return s < 1 ? 1 : (s > max_splits ? max_splits : s);
}

// Forms the items with costs estimated from the tile's position, and their order (the dense baseline).
int run_schedule(const Layer& L, const int* q_cnt, const int* budget, int b_cap, int tile_m, int* sched, hipStream_t st);
int persistent_grid();      // workgroups that fill the device at two per CU

// Called by one thread.  Position in the hand-out order of the next item, or -1 when every queue is drained:
// the workgroup's own queue (its XCD's) while it lasts, then whichever queue has the most items left.  queues = 1: a list
// that is known to be one queue, where nobody should come late because its XCD's is empty (with two workgroups per CU the
// first XCD would take two of the longest items to each of its CUs: fp32 forward, 8 heads, d = 128, 10000 tokens 1380 -> 1210 us).
__device__ __forceinline__ int sched_next(int* __restrict__ sched, int queues = kSchedQueues) {
  const int home = blockIdx.x % queues;
  {
    const int end = sched[kSchedEnd + home];
    if (__atomic_load_n(sched + kSchedCursor + home, __ATOMIC_RELAXED) < end) {
      const int k = atomicAdd(sched + kSchedCursor + home, 1);
      if (k < end) return k;
    }
  }
  for (;;) {                                   // every pass either returns or finds one more queue drained
    int best = -1, left = 0;
    for (int q = 0; q < kSchedQueues; ++q) {
      const int rem = sched[kSchedEnd + q] - __atomic_load_n(sched + kSchedCursor + q, __ATOMIC_RELAXED);
      if (rem > left) left = rem, best = q;
    }
    if (best < 0) return -1;
    const int k = atomicAdd(sched + kSchedCursor + best, 1);
    if (k < sched[kSchedEnd + best]) return k;
  }
}

// hand-out position -> (head index bh, query tile tq)
__host__ __device__ inline void sched_decode(const int* __restrict__ sched, size_t order_off, int k, int& bh, int& tq) {
  const unsigned v = (unsigned)sched[order_off + k];
  bh = (int)(v >> 16);
  tq = (int)(v & 0xffffu);
}

// key tiles streamed by tile tq of a head with nt tiles and nk selected keys, estimated from its position
__host__ __device__ inline int sched_estimate(int tq, int nt, int nk, int causal) {
  if (!causal) return (nk + kTileN - 1) / kTileN;
  const long long keys = ((long long)nk * (tq + 1) + nt - 1) / nt;
  return (int)((keys + kTileN - 1) / kTileN);
}

// head-major item id -> 64-bit sort key, handed out in descending order: queue 0 first, inside a queue the heads in
// the order they were placed, inside a head larger cost first, lower id first among equals.  place = queue << 16 |
// position of the head in its queue (0 for the single list); cost < 2^16 key tiles.
__host__ __device__ inline unsigned long long sched_key(int cost, int id, unsigned place = 0u) {
  const unsigned long long q = 7u - (place >> 16), pos = 0x1fffu - (place & 0x1fffu);
  const unsigned c = cost < 0xffff ? (unsigned)cost : 0xffffu;
  return (q << 61) | (pos << 48) | ((unsigned long long)c << 32) | (unsigned)(0xffffffffu - (unsigned)id);
}

// Placement of the heads on the queues: in order of cost (descending, lower index first among equals) every head
// goes to the least loaded queue (lowest index among equals).  Loads are kept as (load << 3 | queue) in 32 bits so
// that the least loaded queue is one unsigned minimum; head costs are scaled down by `shift` bits to fit.
__host__ __device__ inline int sched_cost_shift(long long total_cost) {
  int shift = 0;
  while ((total_cost >> shift) >= (1ll << 27)) ++shift;
  return shift;
}

// Queues only pay while no head outweighs a queue's fair share by much: the workgroups of the other XCDs come to
// help such a head only when their own queues are drained, and what they then take are its middle-sized items, one
// of which is the tail (per-head budgets on the 64k layer, where one head holds 30 % of the work: 1.68 -> 1.92 ms
// with queues; at 13 % of the work, the shared budget, nothing is lost).  The line is drawn at 1.5 fair shares.
__host__ __device__ inline bool sched_queues_pay(long long total_cost, long long largest_head, int queues) {
  return 2 * largest_head * queues <= 3 * total_cost;
}

// Inside a queue head follows head where a workgroup's share is several times the longest item; elsewhere the long items
// of the last head would start late, and the queue hands out its items longest first, whatever their head (the heads of a
// queue then advance side by side, a few workgroups each).  Attention call, 28 heads, a third of the queries kept: head
// after head against one list 5.50 / 5.65 ms at 64k (a share is 4.6 longest items) but 1.57 / 1.52 at 32k (2.3); longest
// first in the queue against one list 1.435 / 1.459 ms at 32k, 821 / 815 us at 24k, 437 / 445 at 16k, 167 / 171 at 8k.
// `workgroups`: one per CU.
__host__ __device__ inline bool sched_long_enough(long long total_cost, long long largest_item, int workgroups) {
  return 10 * total_cost >= 34 * largest_item * workgroups;
}

// The same list on the host, with estimated costs (diagnostic entry point): the items in hand-out order and the ends of the
// queues.
struct HostWorkList {
  std::vector<int> packed, cost;
  int end[kSchedQueues];
};
HostWorkList sched_build_host(const int* q_cnt, const int* budget, int B, int Hq, int N, int b_cap, int causal, int tile_m,
                              int queues, int workgroups);

}  // namespace omni
