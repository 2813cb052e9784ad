// Selection machinery: k-th largest by radix select over LDS histograms, the
// recall budget search, distribution moments, and ordered stream compaction.
// Serves omni_select_queries (query-mask equation), omni_kv_budget (kurtosis,
// budget equation) and omni_select_kv (key-mask equation).
//
// All decisions are taken on the float32 score arrays through an
// order-preserving map to unsigned keys, so the kept sets are exact functions
// of the input bits.  Sums that decide the budget are accumulated as 64-bit
// fixed point (2^-40 units) with integer atomics: exact, hence independent of
// the order in which lanes arrive.
#include <cmath>
#include <cstring>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace omni {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr double kFixScale = 1099511627776.0;   // 2^40

// a * 2^40 rounded towards zero, 0 for what is not positive, exact: the integer part of a * 2^8 and its fraction times
// 2^32 are both exact in fp32.  (Through fp64 it is three times the instructions, and one workgroup converts a head.)
__device__ __forceinline__ unsigned long long to_fixed(float a) {
  const float x = fmaxf(a, 0.f) * 256.f;
  const unsigned hi = __float2uint_rz(x), lo = __float2uint_rz(__builtin_amdgcn_fractf(x) * 4294967296.f);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ float key_value(unsigned key) {         // inverse of float_key
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// One workgroup finds a cut in a vector of any length: histograms of 2048 bins over an interval of keys that shrinks to the
// bin of the cut, pass by pass.  The first interval is that of a sample (vectors in LDS: of all elements), the two end bins
// taking what lies outside: scores fill a few octaves, and bins of a fixed quarter octave put a third of a head's elements
// on one address of the histogram, which then takes them one after the other.  Only the first pass looks at the whole
// vector; the elements of the bin it picks are copied to LDS, and once no more than kFew are left they are ranked against
// each other.  28 heads, kurtosis + budget + cuts of both lists, as four passes of 8 bits over the whole vector and
// kernels of their own for arg-min, counts, scans and lists (nine launches) / digits of 11, 11 and 10 bits and a kernel for
// the lists / now: 1k scores 53 / 28 / 21 us, 64k 150 / 95 / 77 us; the three calls on scores in hand at 32k 79 -> 60 us.
// What a pass costs beside its sweep is barriers and latencies, 1 to 2 us: hence 256 elements that are ranked against each other
// (64 left one pass more to most vectors beyond 8192) and the first loads of a sweep under the clearing and the picking before it.
// The three calls, before / now: 10451 tokens 55.6 / 51.7 us, 23036 69.5 / 65.3, 48349 96.5 / 91.1.
constexpr int kBins = 2048;
constexpr int kPitch = kBins + 8;       // words between two replicas of the count histogram: other banks for a bin's replicas
constexpr int kReps = 4;                // replicas of a bin, so that lanes on one bin rarely meet on an address
constexpr int kCand = 8192;
constexpr int kFew = 256;               // elements that are ranked against each other, by four threads each, instead of histogrammed
struct __attribute__((aligned(16))) RadixShared {
  union {
    unsigned cnt[kReps * kPitch];
    unsigned long long sum[kReps * kPitch];
  };
  float cand[kCand], few[kFew];
  unsigned few_key[kFew];
  unsigned long long few_mass[kFew];
  unsigned long long wave_tot[kSelWaves];
  unsigned long long rem;
  unsigned key, bin;
  unsigned top, not_bottom;               // range of the sampled keys: the largest, and the complement of the smallest
  int count, found, alone;
};

struct RadixCut {
  bool found;                           // false: the whole vector falls short of the target
  bool alone;                           // mass: the largest element reaches the target by itself, the rest is not set
  unsigned key;                         // the cut: key of the last element taken
  unsigned long long rem;               // count (or mass) still to take among the elements equal to the cut
  unsigned long long other;             // mass (or count) of the elements above the cut
};

__device__ __forceinline__ unsigned long long block_sum(unsigned long long v, RadixShared& sh) {
  v = wave_scan(v);
  __syncthreads();
  if (lane_id() == 63) sh.wave_tot[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long t = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) t += sh.wave_tot[w];
  return t;
}

// The vector x[0, n) by the whole workgroup: f(v) for every kBatch elements of a thread.  Past the end the value is the NaN of
// key 0, below every score, which a histogram may count: a cut never gets down to it.
constexpr int kBatch = 8;               // loads in flight per thread
typedef float Batch[kBatch];
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));      // rows start at any multiple of four bytes
// Element i of a stretch of a head's vector: one 32-bit offset to a base in scalar registers.  Where the stretch begins belongs to the
// base: a vector may be longer than the 2^30 elements that the offset reaches.
template <typename V = float>
__device__ __forceinline__ V element(const float* __restrict__ row, int i) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(row) + (unsigned)i * 4u);
}
// In LDS or in memory, an element per load.  f's second argument: how many of the eight anybody has; the loops end there, because on
// short vectors the fetch of the code, 0.4 us a kilobyte, is a good part of a kernel's time.
template <typename F>
__device__ __forceinline__ void sweep(const float* x, int n, F f) {
#pragma unroll 1
  for (int at = 0; at < n; at += kBatch * kSelThreads) {
    const int some = min(kBatch, cdiv(n - at, kSelThreads));
    Batch v;
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      if (e >= some) break;
      const int o = at + e * kSelThreads + (int)threadIdx.x;
      const float t = x[min(o, n - 1)];
      v[e] = o < n ? t : __uint_as_float(0xffffffffu);
    }
    f(v, some);
  }
}
// In memory, at least four elements: four neighbours per load, the next sixteen elements of a thread in flight under those in hand, and
// the first ones under whatever comes before the sweep (the caller starts them).  Nothing is checked but in the last stretch: a load
// that would pass the end is moved back to it, and of its elements those count that an earlier load does not have.  Bound by the
// vector ALU of the one CU (a few dozen instructions per 64 elements).
constexpr int kLoads = 4, kStep = 4 * kLoads * kSelThreads;
struct Ahead {
  f32x4_any quad[kLoads];
  __device__ __forceinline__ void load(const float* __restrict__ x, int n, int at) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u) quad[u] = element<f32x4_any>(x + min(at, n - 4), min(4 * (u * kSelThreads + (int)threadIdx.x), max(0, n - 4 - at)));
  }
};
template <typename F>
__device__ __forceinline__ void sweep_memory(const float* __restrict__ x, int n, Ahead& next, F f) {
#pragma unroll 1
  for (int at = 0;; at += kStep) {
    const bool more = n - at > kStep;
    Batch v[2];
#pragma unroll
    for (int e = 0; e < 2 * kBatch; ++e) v[e / kBatch][e % kBatch] = next.quad[e / 4][e % 4];
    if (more) {
      next.load(x, n, at + kStep);
    } else {
#pragma unroll
      for (int e = 0; e < 2 * kBatch; ++e) {
        const int i = at + 4 * (e / 4 * kSelThreads + (int)threadIdx.x);
        if (min(i, n - 4) + e % 4 < i) v[e / kBatch][e % kBatch] = __uint_as_float(0xffffffffu);
      }
    }
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      const int some = min(kBatch, 4 * cdiv(n - at - half * kStep / 2, 4 * kSelThreads));
      if (some <= 0) break;
      if (half) {
#pragma unroll
        for (int e = 0; e < kBatch; ++e) v[0][e] = v[1][e];
      }
      f(v[0], some);
    }
    if (!more) return;
  }
}

// Every element in memory, nothing in the place of those past the end.
template <typename F>
__device__ __forceinline__ void sweep_real(const float* __restrict__ x, int n, F f) {
#pragma unroll 1
  for (int at = 0; at < n; at += kBatch * kSelThreads) {
    Batch v;
    const int some = min(kBatch, cdiv(n - at, kSelThreads));
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      if (e >= some) break;
      v[e] = element(x + at, min(e * kSelThreads + (int)threadIdx.x, n - 1 - at));
    }
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      if (e >= some) break;
      if (at + e * kSelThreads + (int)threadIdx.x < n) f(v[e]);
    }
  }
}

template <bool MASS>
__device__ __forceinline__ void histogram_clear(RadixShared& sh, int reps) {
  const int words = reps * kPitch * (MASS ? 2 : 1);
  for (int t = 4 * threadIdx.x; t < words; t += 4 * kSelThreads)
    *reinterpret_cast<u32x4*>(&sh.cnt[t]) = u32x4{0u, 0u, 0u, 0u};
  if (threadIdx.x == 0) sh.found = 0, sh.alone = 0;
}
template <bool MASS>
__device__ __forceinline__ void histogram_add(RadixShared& sh, int rep, unsigned digit, float value) {
  if (MASS) atomicAdd(&sh.sum[rep + digit], to_fixed(value));
  else atomicAdd(&sh.cnt[rep + digit], 1u);
}
// The bin at which the running total from the top reaches sh.rem: into sh.bin, with sh.rem moved on to it.
// Thread t owns the bins 2047 - 2t and 2046 - 2t.  False: the histogram falls short.
template <bool MASS>
__device__ __forceinline__ bool histogram_pick(RadixShared& sh, int reps) {
  __syncthreads();
  unsigned long long c0 = 0, c1 = 0;
  const int pair = kBins / 2 - 1 - (int)threadIdx.x;
#pragma unroll 4
  for (int r = 0; r < reps; ++r) {
    if (MASS) {
      c1 += sh.sum[r * kPitch + 2 * pair];
      c0 += sh.sum[r * kPitch + 2 * pair + 1];
    } else {
      c1 += sh.cnt[r * kPitch + 2 * pair];
      c0 += sh.cnt[r * kPitch + 2 * pair + 1];
    }
  }
  unsigned long long incl = wave_scan(c0 + c1);
  if (lane_id() == 63) sh.wave_tot[threadIdx.x >> 6] = incl;
  const unsigned long long rem = sh.rem;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) incl += w < (int)(threadIdx.x >> 6) ? sh.wave_tot[w] : 0ull;
  const unsigned long long excl = incl - c0 - c1;
  if (excl < rem && rem <= incl) {                                   // one thread at most: its bins hold the crossing
    const bool second = excl + c0 < rem;
    sh.found = 1;
    sh.bin = (unsigned)(kBins - 1 - 2 * (int)threadIdx.x - (second ? 1 : 0));
    sh.rem = rem - excl - (second ? c0 : 0);
  }
  __syncthreads();
  return sh.found;
}

__device__ __forceinline__ unsigned wave_max_unsigned(unsigned v) {        // in lane 63
  v = max(v, dpp_or_zero<0x111, 0xf>(v));
  v = max(v, dpp_or_zero<0x112, 0xf>(v));
  v = max(v, dpp_or_zero<0x114, 0xf>(v));
  v = max(v, dpp_or_zero<0x118, 0xf>(v));
  v = max(v, dpp_or_zero<0x142, 0xa>(v));
  v = max(v, dpp_or_zero<0x143, 0xc>(v));
  return v;
}

// Cut of the vector x[0, n) at `target`: a number of elements (MASS false) or a fixed-point mass (MASS true), largest
// first.  target >= 1.  want_other: whether the cut's `other` is of use.
template <bool MASS>
__device__ RadixCut radix_cut(const float* x, int n, unsigned long long target, bool want_other, RadixShared& sh) {
  // short vectors go to LDS first: the passes over them are then free of memory latencies
  constexpr int kEach = kCand / kSelThreads;
  const bool staged = n <= kCand;
  float sample[kEach];
  if (staged) {
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
      if (e * kSelThreads >= n) break;
      sample[e] = element(x, min(e * kSelThreads + (int)threadIdx.x, n - 1));
    }
  } else {
    sample[0] = x[(long long)n * threadIdx.x / kSelThreads];
  }
  Ahead ahead;
  if (!staged) ahead.load(x, n, 0);
  __syncthreads();
  if (threadIdx.x == 0) {
    sh.rem = target;
    sh.top = sh.not_bottom = 0u;
  }
  unsigned lo = 0u, hi = 0xffffffffu;              // the cut's key is one of these
  const float* src = staged ? sh.cand : x;         // the elements that can still be the cut are among these m
  int m = n, reps = kReps, left = n;
  unsigned long long other = 0;
  float top = 0.f;
#pragma unroll 1
  for (int pass = 0; pass < 4 && lo != hi; ++pass) {         // intervals of at most 2^32, 2^32, 2^21, 2^10 and one key
    histogram_clear<MASS>(sh, reps);
    if (threadIdx.x == 0) sh.count = 0;
    __syncthreads();
    unsigned from = lo, range = hi - lo;           // the bins cover the keys from .. from + range, and more where that is free
    if (pass == 0) {
      unsigned mx = float_key(sample[0]), nmn = ~mx;
      if (staged) {
#pragma unroll
        for (int e = 0; e < kEach; ++e) {
          if (e * kSelThreads >= n) break;
          const unsigned key = float_key(sample[e]);
          mx = max(mx, key);
          nmn = max(nmn, ~key);
          if (e * kSelThreads + (int)threadIdx.x < n) sh.cand[e * kSelThreads + threadIdx.x] = sample[e];
        }
      }
      mx = wave_max_unsigned(mx);
      nmn = wave_max_unsigned(nmn);
      if (lane_id() == 63) {
        atomicMax(&sh.top, mx);
        atomicMax(&sh.not_bottom, nmn);
      }
      __syncthreads();
      from = ~sh.not_bottom;
      range = sh.top - from;
    }
    const int shift = max(0, 21 - __clz((int)range));                  // 32 - 11 significant bits
    auto bin_of = [&](unsigned key) { return key <= from ? 0u : min((key - from) >> shift, (unsigned)kBins - 1); };
    const int rep = ((int)threadIdx.x & (reps - 1)) * kPitch;
    const bool first = pass == 0 && !staged;       // the whole vector, in memory
    if (first) {
      sweep_memory(x, n, ahead, [&](const Batch& v, int some) {
#pragma unroll
        for (int e = 0; e < kBatch; ++e) {
          if (e >= some) break;
          histogram_add<MASS>(sh, rep, bin_of(float_key(v[e])), v[e]);
          if (MASS) top = fmaxf(top, v[e]);
        }
      });
    } else {
      sweep(src, m, [&](const Batch& v, int some) {
#pragma unroll
        for (int e = 0; e < kBatch; ++e) {
          if (e >= some) break;
          const unsigned key = float_key(v[e]);
          if (key - lo <= hi - lo) histogram_add<MASS>(sh, rep, bin_of(key), v[e]);
          if (MASS) top = fmaxf(top, v[e]);
        }
      });
    }
    if (first) ahead.load(x, n, 0);
    // infinite and huge elements: the sums may have left 64 bits
    if (MASS && (top >= 16777216.f || to_fixed(top) >= target)) sh.alone = 1;
    const bool found = histogram_pick<MASS>(sh, reps);
    if (MASS && sh.alone) return RadixCut{true, true, 0u, 0ull, 0ull};
    if (!found) return RadixCut{false, false, 0u, 0ull, 0ull};                                  // first pass only
    // What lies above the bin is taken whole, what lies in it is copied to LDS as far as it fits: the first time to the
    // long list, from there to the short one.
    const unsigned bin = sh.bin;
    const unsigned long long begin = (unsigned long long)from + ((unsigned long long)bin << shift), end = begin + (1ull << shift) - 1;
    const unsigned before = hi, lo1 = bin == 0u ? lo : (unsigned)begin;
    hi = bin == kBins - 1u || end > hi ? hi : (unsigned)end;
    lo = lo1;
    float* list = src == sh.cand ? sh.few : sh.cand;
    const int cap = src == sh.cand ? kFew : kCand;
    auto part = [&](const Batch& v, int some) {
      unsigned mine = 0;
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        if (e >= some) break;
        const unsigned key = float_key(v[e]);
        const bool over = key > hi && key <= before;
        mine |= key - lo <= hi - lo ? 1u << e : 0u;
        if (MASS) other += over;
        else if (want_other) other += over ? to_fixed(v[e]) : 0ull;    // a third of the sweep's instructions
      }
      if (!__any(mine)) return;
      const unsigned n_mine = __popc(mine), incl = wave_scan(n_mine);
      int at = 0;
      if (lane_id() == 63) at = atomicAdd(&sh.count, (int)incl);
      at = __builtin_amdgcn_readlane(at, 63) + (int)(incl - n_mine);
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        if (e >= some) break;
        if (mine >> e & 1u) {
          if (at < cap) list[at] = v[e];
          ++at;
        }
      }
    };
    if (first) sweep_memory(x, n, ahead, part);
    else sweep(src, m, part);
    __syncthreads();
    left = sh.count;
    if (left <= cap) {
      src = list;
      m = left;
      reps = 1;
    }
    if (left <= kFew) break;
    __syncthreads();                               // sh.count is set again
  }
  if (threadIdx.x == 0) sh.key = lo;
  if (left <= kFew && lo != hi) {
    // Every element left against every other, by four lanes: the one whose own share crosses sh.rem is the cut (equal elements
    // all write the same values).
    const float* few = src;                        // the short list, or the long one where that was enough
    const unsigned long long rem = sh.rem;
    __syncthreads();
    if ((int)threadIdx.x < left) {
      const float own = few[threadIdx.x];
      sh.few_key[threadIdx.x] = float_key(own);
      sh.few_mass[threadIdx.x] = to_fixed(own);
    }
    __syncthreads();
    const int who = (int)threadIdx.x >> 2;
    unsigned mine = 0;
    if (who < left) {
      mine = sh.few_key[who];
      unsigned more = 0, same = 0;
      unsigned long long mass = 0;
#pragma unroll 8
      for (int t = (int)threadIdx.x & 3; t < left; t += 4) {
        const unsigned k = sh.few_key[t];
        more += k > mine;
        same += k == mine;
        if (MASS) mass += k > mine ? sh.few_mass[t] : 0ull;
      }
#pragma unroll
      for (int o = 1; o < 4; o <<= 1) {
        more += __shfl_xor(more, o, 4);
        same += __shfl_xor(same, o, 4);
        if (MASS) mass += __shfl_xor(mass, o, 4);
      }
      const unsigned long long excl = MASS ? mass : more, own = MASS ? same * sh.few_mass[who] : same;
      if (excl < rem && rem <= excl + own) {
        sh.key = mine;
        sh.rem = rem - excl;
      }
    }
    __syncthreads();
    if (who < left && ((int)threadIdx.x & 3) == 0 && mine > sh.key) other += MASS ? 1ull : sh.few_mass[who];
  }
  other = block_sum(other, sh);
  const RadixCut cut{true, false, sh.key, sh.rem, other};
  __syncthreads();                                 // sh may be used again
  return cut;
}

// Membership rule of a list.
struct KeepRule {
  int keep_all_head0;    // head 0 keeps everything
  int visual_only;       // only the visual range is classified, elements outside are always kept (queries)
  int use_table;         // thresholds from thr/need arrays, else from thr_scalar with need 0
  unsigned thr_scalar;
};

// One list to form: the scores, the rule, the cut of every head and what comes out.
struct ListJob {
  const float* x;        // [B*H, ld]
  KeepRule rule;
  unsigned* thr;         // [B*H] the cut, from the kernel that finds it for the one that writes the list (long vectors)
  int* need;             // [B*H]
  int* off_keep;         // [B*H, nchunk] and the elements always taken, and those at the cut, before each chunk of kChunk
  int* off_eq;           // elements
  int* out;              // [B*H, out_stride], or null: no list
  int out_stride;
  int* total;            // [B*H] length of the list, or null
};

// Cut of a head's own budget, as the budget search leaves it: elements above `key` and `need` of those at it.
// need < 0: not known (the whole vector, or one element that is infinite or beyond the fixed point).
struct OwnCut {
  unsigned* key;         // [B*H]
  int* need;             // [B*H]
};
__device__ __forceinline__ float recall_of(unsigned long long mass, int N) {
  return (float)((double)mass / kFixScale / (double)(float)N);
}

// How many elements each head of a job takes.
struct KeySource {
  int mode;              // 0: budget of the flattest head, 1: largest budget of the heads, 2: the head's own (all from
                         // own[B*H] and kurt), 3: given counts (budget array), 4: top fraction of the visual range
  const int* own;        // [B*H] budget of every head's own scores
  OwnCut cut;            // and the cut that this budget makes, or null; for long vectors this is the job's own thr and need
  const double* kurt;    // [B*H]
  int* flattest;         // [B] out (modes 0..2)
  int* budget;           // [B] or [B*H] out (modes 0..2), in (mode 3)
  int bph, k_cap;
  float fraction;
  float* recall;         // [B*H] out or null
};

__device__ __forceinline__ void classify(const KeepRule& r, int h, bool inside, float v, unsigned thr, bool& always,
                                         bool& eq) {
  if ((r.keep_all_head0 && h == 0) || (r.visual_only && !inside)) {
    always = true;
    eq = false;
    return;
  }
  const unsigned key = float_key(v);
  always = key > thr;
  eq = key == thr;
}

// ------------------------------------------------------------------ kernels

// Wavefront-wide argmin over the heads' kurtoses: heads within 1e-9 (relative) of the smallest tie and the lowest index
// wins (for two or three scores the statistic is one constant for every head and rounding would pick the head).
__device__ __forceinline__ int flattest_head(const double* __restrict__ kurt, int H) {
  double v = kurt[0];
  for (int h = lane_id(); h < H; h += 64) v = fmin(v, kurt[h]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  const double bar = v + 1e-9 * fabs(v);
  for (int h0 = 0; h0 < H; h0 += 64) {
    const int h = h0 + lane_id();
    const unsigned long long bal = __ballot(h < H && kurt[h] <= bar);
    if (bal) return h0 + __ffsll((long long)bal) - 1;
  }
  return H - 1;
}

// grid: (H, B, 2).  Of every head's own scores: excess kurtosis m4/m2^2 - 3 in fp64 with a fixed reduction tree (z = 0),
// and the smallest count whose largest elements reach recall_p of the mass (z = 1).  Every head finds its budget
// although the shared budget needs the flattest head's only: the heads run side by side, and the search does not wait
// for the arg-min.
// only_flattest: grid (1, B), the budget of every sequence's flattest head, after a launch of (H, B, 1) (see launch_stats).
__global__ __launch_bounds__(kSelThreads) void score_stats_kernel(const float* __restrict__ a, Layer L, Ragged rg,
                                                                 double recall_p, int only_flattest,
                                                                 double* __restrict__ kurt, int* __restrict__ own,
                                                                 OwnCut own_cut, float* __restrict__ recall) {
  __shared__ RadixShared sh;
  __shared__ double red[2][kSelWaves];
  const int b = blockIdx.y, head = only_flattest ? flattest_head(kurt + (long long)b * L.Hq, L.Hq) : (int)blockIdx.x;
  const int bh = b * L.Hq + __builtin_amdgcn_readfirstlane(head);
  const int N = seq_len(L, rg, b);
  const float* x = a + (long long)bh * L.ld;
  if (blockIdx.z || only_flattest) {
    // rounded up: the truncated element masses must never reach a target below the real one
    const unsigned long long target = (unsigned long long)ceil(recall_p * (double)N * kFixScale);
    const RadixCut cut = radix_cut<true>(x, N, target, true, sh);
    if (threadIdx.x == 0) {
      int r = N;                                // even the whole vector falls short: take everything
      unsigned at = 0u;
      int need = -1;
      if (cut.alone) {
        r = 1;
      } else if (cut.found) {
        const unsigned long long v = to_fixed(key_value(cut.key)), q = (cut.rem + v - 1) / v;   // v > 0: its bin crossed the target
        r = max(1, (int)min((unsigned long long)N, cut.other + q));
        if (cut.other + q == (unsigned long long)r && r < N) {
          at = cut.key;
          need = (int)q;
          if (recall) recall[bh] = recall_of(target - cut.rem + q * v, N);
        }
      }
      own[bh] = r;
      own_cut.key[bh] = at;
      own_cut.need[bh] = need;
    }
    return;
  }
  const int w = threadIdx.x >> 6;
  double s = 0.0;
  sweep_real(x, N, [&](float v) { s += (double)v; });
  s = wave_sum(s);
  if (lane_id() == 0) red[0][w] = s;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < kSelWaves; ++i) t += red[0][i];
  const double mu = t / (double)N;
  double s2 = 0.0, s4 = 0.0;
  sweep_real(x, N, [&](float v) {
    const double c = (double)v - mu, c2 = c * c;
    s2 += c2;
    s4 += c2 * c2;
  });
  s2 = wave_sum(s2);
  s4 = wave_sum(s4);
  __syncthreads();
  if (lane_id() == 0) {
    red[0][w] = s2;
    red[1][w] = s4;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t2 = 0.0, t4 = 0.0;
#pragma unroll
    for (int i = 0; i < kSelWaves; ++i) {
      t2 += red[0][i];
      t4 += red[1][i];
    }
    const double m2 = t2 / (double)N, m4 = t4 / (double)N;
    kurt[bh] = m2 > 0.0 ? m4 / (m2 * m2) - 3.0 : -2.0;
  }
}

constexpr int kSpan = 8 * kSelThreads;   // elements of a vector whose list the workgroup that finds the cut writes itself
struct ListShared {
  int keep[kSelWaves], eq[kSelWaves];
};
// The list of a vector of at most kSpan elements, ascending: every wavefront holds up to 512 neighbours and ranks them by 64-bit
// masks.
__device__ __forceinline__ void short_list(const ListJob& job, const float* __restrict__ row, int h, int bh, int N, int v0, int v1,
                                           unsigned thr, int need, ListShared& sh) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = lane_id();
  const bool all = job.rule.keep_all_head0 && h == 0;
  const int lo = all ? N : job.rule.visual_only ? v0 : 0, hi = all ? N : job.rule.visual_only ? v1 : N;
  // elements outside [lo, hi) are always taken, those inside by the cut
  const int blocks = cdiv(N, kSelThreads);                 // of 64 elements, for each wavefront
  const int own = w * blocks * 64;
  float v[kSpan / kSelThreads];
#pragma unroll
  for (int e = 0; e < kSpan / kSelThreads; ++e) {
    if (e >= blocks) break;
    v[e] = element(row, min(own + e * 64 + lane, N - 1));
  }
  // of the 64 elements from n0 on: those always taken, those at the cut
  const bool plain = own >= lo && own + blocks * 64 <= hi;
  auto masks = [&](int n0, float x, unsigned long long& above, unsigned long long& at_cut) {
    const unsigned key = float_key(x);
    if (plain) {
      above = __ballot(key > thr);
      at_cut = __ballot(key == thr);
    } else {
      const int n = n0 + lane;
      const bool real = n < N, free = n < lo || n >= hi;
      above = __ballot(real && (free || key > thr));
      at_cut = __ballot(real && !free && key == thr);
    }
  };
  int keep = 0, eq = 0;
#pragma unroll
  for (int e = 0; e < kSpan / kSelThreads; ++e) {
    if (e >= blocks) break;
    unsigned long long above, at_cut;
    masks(own + e * 64, v[e], above, at_cut);
    keep += (int)__popcll(above);
    eq += (int)__popcll(at_cut);
  }
  if (lane == 0) {
    sh.keep[w] = keep;
    sh.eq[w] = eq;
  }
  __syncthreads();
  int pk = 0, pe = 0, all_k = 0, all_e = 0;                // before this wavefront's elements, in all
#pragma unroll
  for (int i = 0; i < kSelWaves; ++i) {
    const int k = sh.keep[i], e = sh.eq[i];
    pk += i < w ? k : 0;
    pe += i < w ? e : 0;
    all_k += k;
    all_e += e;
  }
  if (threadIdx.x == 0 && job.total) job.total[bh] = min(job.out_stride, all_k + min(all_e, need));
  const auto below = [](unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
  };
  int* dst = job.out + (long long)bh * job.out_stride;
#pragma unroll
  for (int e = 0; e < kSpan / kSelThreads; ++e) {
    const int n0 = own + e * 64;
    if (e >= blocks) break;
    unsigned long long above, at_cut;
    masks(n0, v[e], above, at_cut);
    int pos = pk + below(above) + min(pe, need);
    bool take = above >> lane & 1ull;
    if (at_cut) {
      const int q = pe + below(at_cut);
      pos += min(q, need) - min(pe, need);
      take = take || ((at_cut >> lane & 1ull) && q < need);
    }
    if (take && pos < job.out_stride) dst[pos] = n0 + lane;
    pk += (int)__popcll(above);
    pe += (int)__popcll(at_cut);
  }
}

constexpr int kChunk = 1024;            // elements per workgroup of the list writer
constexpr int kChunkThreads = 256;
constexpr int kPerThread = kChunk / kChunkThreads;
// Longer vectors: the counts before every chunk; a wavefront counts a chunk at a time.
__device__ __forceinline__ void chunk_counts(const ListJob& job, const float* __restrict__ row, int h, int bh, int N, int stride,
                                             int v0, int v1, unsigned thr, int need) {
  const int lane = lane_id(), nchunk = cdiv(N, kChunk);
  const bool all = job.rule.keep_all_head0 && h == 0;
  const int lo = job.rule.visual_only ? v0 : 0, hi = job.rule.visual_only ? v1 : N;
  int* ck = job.off_keep + (long long)bh * stride;
  int* ce = job.off_eq + (long long)bh * stride;
  if (all) {                               // nothing to look at
    for (int c = threadIdx.x; c < nchunk; c += kSelThreads) {
      ck[c] = c * kChunk;
      ce[c] = 0;
    }
    if (threadIdx.x == 0 && job.total) job.total[bh] = min(job.out_stride, N);
    return;
  }
#pragma unroll 1
  for (int c = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); c < nchunk; c += kSelWaves) {
    float v[kChunk / 64];
#pragma unroll
    for (int e = 0; e < kChunk / 64; ++e) v[e] = element(row + c * kChunk, min(e * 64 + lane, N - 1 - c * kChunk));
    unsigned above = 0, at_cut = 0;
    if (c * kChunk >= lo && (c + 1) * kChunk <= hi) {
#pragma unroll
      for (int e = 0; e < kChunk / 64; ++e) {
        const unsigned key = float_key(v[e]);
        above += key > thr;
        at_cut += key == thr;
      }
    } else {
#pragma unroll
      for (int e = 0; e < kChunk / 64; ++e) {
        const int n = c * kChunk + e * 64 + lane;
        const unsigned key = float_key(v[e]);
        const bool real = n < N, free = n < lo || n >= hi;
        above += real && (free || key > thr);
        at_cut += real && !free && key == thr;
      }
    }
    const unsigned both = wave_scan(above | at_cut << 16);
    if (lane == 63) {
      ck[c] = (int)(both & 0xffffu);
      ce[c] = (int)(both >> 16);
    }
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  int run_k = 0, run_e = 0;
  for (int c0 = 0; c0 < nchunk; c0 += 64) {
    const int c = c0 + lane;
    const unsigned vk = c < nchunk ? ck[c] : 0, ve = c < nchunk ? ce[c] : 0;
    const unsigned sk = wave_scan(vk), se = wave_scan(ve);
    if (c < nchunk) {
      ck[c] = run_k + (int)(sk - vk);
      ce[c] = run_e + (int)(se - ve);
    }
    run_k += __builtin_amdgcn_readlane((int)sk, 63);
    run_e += __builtin_amdgcn_readlane((int)se, 63);
  }
  if (lane == 0 && job.total) job.total[bh] = min(job.out_stride, run_k + min(run_e, need));
}

// grid: (H, B, jobs).  Per head: how many elements to take, the cut (threshold key, number of cut-valued elements to
// take), the recall.  Vectors of one span: and the list, which a launch of its own (list_write_kernel) writes otherwise.
__global__ __launch_bounds__(kSelThreads) void list_cut_kernel(Layer L, Ragged rg, ListJob job0, KeySource src0,
                                                              ListJob job1, KeySource src1) {
  __shared__ RadixShared sh;
  __shared__ ListShared lsh;
  __shared__ int k_sh;
  const ListJob& job = blockIdx.z ? job1 : job0;
  const KeySource& src = blockIdx.z ? src1 : src0;
  const int H = L.Hq, h = blockIdx.x, b = blockIdx.y, bh = b * H + h;
  const int N = seq_len(L, rg, b), v0 = rg.on ? rg.v0[b] : L.v0, v1 = rg.on ? rg.v1[b] : L.v1;
  const float* row = job.x + (long long)bh * L.ld;
  unsigned thr = job.rule.thr_scalar;
  int need = 0;
  if (job.rule.use_table) {
    if (src.mode <= 2 && threadIdx.x < 64) {
      const int flat = flattest_head(src.kurt + (long long)b * H, H);
      int k;
      if (src.mode == 0) {
        k = src.own[b * H + flat];
      } else if (src.mode == 1) {
        k = 0;
        for (int i = threadIdx.x; i < H; i += 64) k = max(k, src.own[b * H + i]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) k = max(k, __shfl_xor(k, o, 64));
      } else {
        k = src.own[bh];
      }
      if (threadIdx.x == 0) {
        k_sh = k;
        if (h == 0) src.flattest[b] = flat;
        if (src.mode == 2) src.budget[bh] = k;
        else if (h == 0) src.budget[b] = k;
      }
    }
    __syncthreads();
    int lo = 0, hi = N;
    long long k;
    if (src.mode <= 2) {
      k = min(k_sh, src.k_cap);
    } else if (src.mode == 3) {
      k = min(src.budget[budget_slot(src.bph, b, bh)], src.k_cap);
    } else {
      lo = v0, hi = v1;
      k = (long long)ceil((double)src.fraction * (double)(v1 - v0));
      k = k < 0 ? 0 : k;
    }
    const int n = hi - lo;
    unsigned long long mass = 0;
    const bool known = src.mode <= 2 && src.cut.need && k == src.own[bh] && src.cut.need[bh] >= 0;     // found by the search for the
    if (known) {                                                                                  // budget, with its recall
      thr = src.cut.key[bh];
      need = src.cut.need[bh];
    } else if ((job.rule.keep_all_head0 && h == 0) || k >= n) {
      thr = 0u;
      if (src.recall) {
        unsigned long long local = 0;
        sweep_real(row + lo, n, [&](float v) { local += to_fixed(v); });
        mass = block_sum(local, sh);
      }
    } else if (k <= 0) {
      thr = 0xffffffffu;
    } else {
      const RadixCut cut = radix_cut<false>(row + lo, n, k, src.recall != nullptr, sh);
      thr = cut.key;
      need = (int)cut.rem;
      mass = cut.other + cut.rem * to_fixed(key_value(cut.key));
    }
    if (threadIdx.x == 0 && src.recall && !known) src.recall[bh] = recall_of(mass, N);
  }
  if (!job.out) return;
  if (L.N <= kSpan) {
    short_list(job, row, h, bh, N, v0, v1, thr, need, lsh);
    return;
  }
  __syncthreads();                      // the cut of the head's own budget, read above, lies where this one goes
  if (threadIdx.x == 0) {
    job.thr[bh] = thr;
    job.need[bh] = need;
  }
  chunk_counts(job, row, h, bh, N, cdiv(L.N, kChunk), v0, v1, thr, need);
}

// grid: (nchunk, B*H, jobs).  Writes the kept indices of the chunk, ascending, at their global rank.
__global__ __launch_bounds__(kChunkThreads) void list_write_kernel(Layer L, Ragged rg, ListJob job0, ListJob job1) {
  __shared__ int wsum[2][kChunkThreads / 64];
  const ListJob job = blockIdx.z ? job1 : job0;
  const int bh = blockIdx.y, h = bh % L.Hq, b = bh / L.Hq;
  const int N = seq_len(L, rg, b), v0 = rg.on ? rg.v0[b] : L.v0, v1 = rg.on ? rg.v1[b] : L.v1;
  if (blockIdx.x * kChunk >= N) return;
  const unsigned thr = job.rule.use_table ? job.thr[bh] : job.rule.thr_scalar;
  const int need = job.rule.use_table ? job.need[bh] : 0;
  const float* row = job.x + (long long)bh * L.ld;
  const int base = blockIdx.x * kChunk + threadIdx.x * kPerThread;
  bool al[kPerThread], eq[kPerThread];
  int ck = 0, ce = 0;
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int n = base + e;
    al[e] = false;
    eq[e] = false;
    if (n < N) classify(job.rule, h, n >= v0 && n < v1, row[n], thr, al[e], eq[e]);
    ck += al[e];
    ce += eq[e];
  }
  // exclusive scan of (ck, ce) over the workgroup
  const int lane = lane_id(), w = threadIdx.x >> 6;
  int sk = ck, se = ce;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int tk = __shfl_up(sk, o, 64);
    const int te = __shfl_up(se, o, 64);
    if (lane >= o) {
      sk += tk;
      se += te;
    }
  }
  if (lane == 63) {
    wsum[0][w] = sk;
    wsum[1][w] = se;
  }
  __syncthreads();
  const long long off = (long long)bh * cdiv(L.N, kChunk) + blockIdx.x;
  int pk = job.off_keep[off] + sk - ck;
  int pe = job.off_eq[off] + se - ce;
  for (int i = 0; i < w; ++i) {
    pk += wsum[0][i];
    pe += wsum[1][i];
  }
  int* dst = job.out + (long long)bh * job.out_stride;
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const bool take = al[e] || (eq[e] && pe < need);
    if (take) {
      const int pos = pk + min(pe, need);
      if (pos < job.out_stride) dst[pos] = base + e;
    }
    pk += al[e];
    pe += eq[e];
  }
}

// grid: B*H.  The sub-range of an ascending index list that lies in [v0, v1).
__global__ void visual_subset_kernel(const int* __restrict__ kv_idx, const int* __restrict__ budget, int bph, int H, int b_cap,
                                     int v0, int v1, int* __restrict__ vis_idx, int* __restrict__ vis_cnt) {
  __shared__ int range[2];
  const int bh = blockIdx.x, b = bh / H;
  const int* src = kv_idx + (long long)bh * b_cap;
  const int n = min(budget[budget_slot(bph, b, bh)], b_cap);
  if (threadIdx.x < 2) {
    const int target = threadIdx.x == 0 ? v0 : v1;      // first position with index >= target
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (src[mid] < target) lo = mid + 1; else hi = mid;
    }
    range[threadIdx.x] = lo;
  }
  __syncthreads();
  const int first = range[0], cnt = range[1] - range[0];
  for (int t = threadIdx.x; t < cnt; t += blockDim.x) vis_idx[(long long)bh * b_cap + t] = src[first + t];
  if (threadIdx.x == 0) vis_cnt[bh] = cnt;
}

struct CutWs {
  unsigned* thr;
  int* need;
  int* cnt_keep;
  int* cnt_eq;
};
CutWs carve_cut(Arena& a, const Layer& L) {
  CutWs w;
  w.thr = a.take<unsigned>((size_t)L.B * L.Hq);
  w.need = a.take<int>((size_t)L.B * L.Hq);
  const size_t chunks = L.N > kSpan ? (size_t)L.B * L.Hq * cdiv(L.N, kChunk) : 0;
  w.cnt_keep = a.take<int>(chunks);
  w.cnt_eq = a.take<int>(chunks);
  return w;
}

ListJob list_job(const CutWs& w, const float* x, const KeepRule& rule, int* out, int out_stride, int* total) {
  ListJob j;
  j.x = x;
  j.rule = rule;
  j.thr = w.thr;
  j.need = w.need;
  j.off_keep = w.cnt_keep;
  j.off_eq = w.cnt_eq;
  j.out = out;
  j.out_stride = out_stride;
  j.total = total;
  return j;
}

ListJob query_job(const Layer& L, const CutWs& w, const float* scores, int mode, float param, int* q_idx, int* q_cnt,
                  KeySource* src) {
  KeepRule rule = {1, 1, mode != 0, 0u};
  if (mode == 0) {
    unsigned u;
    std::memcpy(&u, &param, 4);
    rule.thr_scalar = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  }
  *src = KeySource{};
  src->mode = 4;
  src->fraction = param;
  return list_job(w, scores, rule, q_idx, L.ld, q_cnt);
}

KeepRule key_rule() { return KeepRule{0, 0, 1, 0u}; }

// The cuts and the lists of one or two jobs: in one launch where a vector is short, else the lists in a launch of their own with a
// workgroup per kChunk elements.  28 heads, both lists, one launch / two: 1072 scores 12.7 us / 16.3, 65536: 64 / 48.  At the line, a
// workgroup a CU, the cuts of many heads run in rounds and the lists with them; omni_select_queries, one launch / two: 8192 scores, 28
// heads 17.5 us / 20.2, 252 21.3 / 25.8, 280 31.0 / 34.0, 448 31.7 / 36.7, 896 58.4 / 66.9; 4096 scores, 896 heads 45.9 / 52.0.
int launch_lists(const Layer& L, const Ragged& rg, int jobs, const ListJob& j0, const KeySource& s0, const ListJob& j1,
                 const KeySource& s1, hipStream_t st) {
  hipLaunchKernelGGL(list_cut_kernel, dim3(L.Hq, L.B, jobs), dim3(kSelThreads), 0, st, L, rg, j0, s0, j1, s1);
  OMNI_LAUNCH_CHECK();
  if (L.N > kSpan && j0.out) {
    hipLaunchKernelGGL(list_write_kernel, dim3(cdiv(L.N, kChunk), L.B * L.Hq, jobs), dim3(kChunkThreads), 0, st, L, rg, j0, j1);
    OMNI_LAUNCH_CHECK();
  }
  return OMNI_OK;
}

// A shared budget (mode 0) needs the flattest head's own only.  While the heads are fewer than the CUs the search of all of
// them beside the kurtoses costs nothing and saves a launch; with more it is work that nobody asked for.  Both lists, all heads /
// the flattest in a launch of its own, us: 4 sequences of 28 heads, 8192 tokens 60.5 / 68.4, 8 69.6 / 72.3, 12 (4096 tokens)
// 107.8 / 104.7, 32 240 / 220, 64 (2048 tokens) 362 / 305.
constexpr int kBudgetHeads = 256;

struct StatsWs {
  int* own;
  OwnCut cut;
};
StatsWs carve_stats(Arena& a, const Layer& L) {
  StatsWs w;
  w.own = a.take<int>((size_t)L.B * L.Hq);
  w.cut.key = a.take<unsigned>((size_t)L.B * L.Hq);
  w.cut.need = a.take<int>((size_t)L.B * L.Hq);
  return w;
}

// kurtosis and own budgets of all heads, and where the counts of the key lists come from
int launch_stats(const Layer& L, const Ragged& rg, const float* key_scores, float recall_p, int budget_mode, double* kurt,
                 const StatsWs& w, int* flattest, int* budget, float* recall, int k_cap, KeySource* src, hipStream_t st) {
  const bool after = budget_mode == 0 && L.B * L.Hq > kBudgetHeads;
  hipLaunchKernelGGL(score_stats_kernel, dim3(L.Hq, L.B, after ? 1 : 2), dim3(kSelThreads), 0, st, key_scores, L, rg,
                     (double)recall_p, 0, kurt, w.own, w.cut, recall);
  OMNI_LAUNCH_CHECK();
  if (after) {
    hipLaunchKernelGGL(score_stats_kernel, dim3(1, L.B), dim3(kSelThreads), 0, st, key_scores, L, rg, (double)recall_p, 1, kurt,
                       w.own, w.cut, recall);
    OMNI_LAUNCH_CHECK();
  }
  *src = KeySource{};
  src->mode = budget_mode;
  src->own = w.own;
  src->cut = after ? OwnCut{} : w.cut;             // known for every head only where all were searched
  src->kurt = kurt;
  src->flattest = flattest;
  src->budget = budget;
  src->k_cap = k_cap;
  src->recall = recall;
  return OMNI_OK;
}

}  // namespace

size_t select_ws(const Layer& L) {
  Arena a(nullptr);
  carve_cut(a, L);
  return a.used();
}

int run_select_queries(const Layer& L, const float* scores, int mode, float param, int* q_idx, int* q_cnt, void* ws,
                       hipStream_t st) {
  Arena a(ws);
  KeySource src;
  const ListJob job = query_job(L, carve_cut(a, L), scores, mode, param, q_idx, q_cnt, &src);
  return launch_lists(L, Ragged{}, 1, job, src, job, src, st);
}

int run_select_kv(const Layer& L, const float* key_scores, const int* budget, int b_cap, int* kv_idx, void* ws,
                  hipStream_t st) {
  Arena a(ws);
  const ListJob job = list_job(carve_cut(a, L), key_scores, key_rule(), kv_idx, b_cap, nullptr);
  KeySource src{};
  src.mode = 3;
  src.budget = const_cast<int*>(budget);
  src.bph = L.bph;
  src.k_cap = b_cap;
  return launch_lists(L, Ragged{}, 1, job, src, job, src, st);
}

size_t budget_stats_ws(const Layer& L) {
  Arena a(nullptr);
  carve_stats(a, L);
  return a.used();
}

int run_budget_stats(const Layer& L, const float* key_scores, float recall_p, int budget_mode, double* kurt,
                     int* flattest, int* budget, float* recall, void* ws, hipStream_t st) {
  Arena a(ws);
  KeySource src;
  const int rc = launch_stats(L, Ragged{}, key_scores, recall_p, budget_mode, kurt, carve_stats(a, L), flattest, budget, recall,
                              L.N, &src, st);
  if (rc != OMNI_OK) return rc;
  const ListJob job = list_job(CutWs{}, key_scores, key_rule(), nullptr, 0, nullptr);   // the cut for the recall only: no list
  return launch_lists(L, Ragged{}, 1, job, src, job, src, st);
}

size_t select_lists_ws(const Layer& L) {
  Arena a(nullptr);
  carve_cut(a, L);
  carve_cut(a, L);
  a.take<int>((size_t)L.B * L.Hq);
  return a.used();
}

int run_select_lists(const Layer& L, const Ragged& rg, const float* scores, int q_mode, float q_param, int* q_idx,
                     int* q_cnt, const float* key_scores, float recall_p, int budget_mode, double* kurt, int* flattest,
                     int* budget, float* recall, int* kv_idx, int b_cap, void* ws, hipStream_t st) {
  Arena a(ws);
  KeySource ks, qs;
  const CutWs kw = carve_cut(a, L), qw = carve_cut(a, L);
  const StatsWs stats = {a.take<int>((size_t)L.B * L.Hq), {kw.thr, kw.need}};
  const int rc = launch_stats(L, rg, key_scores, recall_p, budget_mode, kurt, stats, flattest, budget, recall, b_cap, &ks, st);
  if (rc != OMNI_OK) return rc;
  const ListJob kj = list_job(kw, key_scores, key_rule(), kv_idx, b_cap, nullptr);
  const ListJob qj = query_job(L, qw, scores, q_mode, q_param, q_idx, q_cnt, &qs);
  return launch_lists(L, rg, 2, qj, qs, kj, ks, st);
}

// ---- union of the stored visual rows over the heads of a KV group, with a membership bit per head
// (paper Sec. "KV Cache Slimming": per-head token-level storage; under grouped-query attention the heads
// of a group index one shared cache, so the group's union is what a decode step can touch at all)

__global__ void fill_u32_kernel(unsigned* p, long long n, unsigned v) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// grid: (cdiv(b_cap, 256), B*Hq)
__global__ void group_mark_kernel(const int* __restrict__ kv_idx, const int* __restrict__ budget, int bph, int Hq, int Hkv, int b_cap,
                                  int v0, int v1, unsigned* __restrict__ umask) {
  const int bh = blockIdx.y, b = bh / Hq, i = bh % Hq, G = Hq / Hkv, g = i / G;
  const int n = min(budget[budget_slot(bph, b, bh)], b_cap);
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int tok = kv_idx[(long long)bh * b_cap + t];
  if (tok < v0 || tok >= v1) return;
  atomicOr(&umask[(long long)(b * Hkv + g) * (v1 - v0) + (tok - v0)], 1u << (i % G));
}

// grid: B*Hkv, 1024 threads.  Ordered compaction of the marked tokens.
__global__ __launch_bounds__(1024) void group_compact_kernel(const unsigned* __restrict__ umask, int nv, int v0, int u_cap,
                                                             int* __restrict__ grp_idx, unsigned* __restrict__ grp_mask,
                                                             int* __restrict__ grp_cnt) {
  __shared__ int wave_cnt[16];
  __shared__ int base;
  const int bg = blockIdx.x;
  const unsigned* src = umask + (long long)bg * nv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) base = 0;
  __syncthreads();
  for (int c0 = 0; c0 < nv; c0 += 1024) {
    const int t = c0 + threadIdx.x;
    const unsigned m = t < nv ? src[t] : 0u;
    const unsigned long long bal = __ballot(m != 0u);
    if (lane == 0) wave_cnt[wave] = __popcll(bal);
    __syncthreads();
    int off = base;
    for (int w = 0; w < wave; ++w) off += wave_cnt[w];
    off += __popcll(bal & ((1ull << lane) - 1ull));
    if (m != 0u && off < u_cap) {
      grp_idx[(long long)bg * u_cap + off] = v0 + t;
      grp_mask[(long long)bg * u_cap + off] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int tot = 0;
      for (int w = 0; w < 16; ++w) tot += wave_cnt[w];
      base += tot;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) grp_cnt[bg] = base;
}

size_t group_subset_ws(const Layer& L) {
  Arena a(nullptr);
  a.take<unsigned>((size_t)L.B * L.Hkv * (L.v1 - L.v0));
  return a.used();
}

int run_group_subset(const Layer& L, const int* kv_idx, const int* budget, int b_cap, int* grp_idx, unsigned* grp_mask,
                     int* grp_cnt, int u_cap, void* ws, hipStream_t st) {
  Arena a(ws);
  const int nv = L.v1 - L.v0;
  const long long n = (long long)L.B * L.Hkv * nv;
  unsigned* umask = a.take<unsigned>((size_t)n);
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)std::min<long long>(cdiv(n, 256LL), 4096)), dim3(256), 0, st, umask, n,
                     0u);
  OMNI_LAUNCH_CHECK();
  hipLaunchKernelGGL(group_mark_kernel, dim3(cdiv(b_cap, 256), L.B * L.Hq), dim3(256), 0, st, kv_idx, budget, L.bph, L.Hq, L.Hkv,
                     b_cap, L.v0, L.v1, umask);
  OMNI_LAUNCH_CHECK();
  hipLaunchKernelGGL(group_compact_kernel, dim3(L.B * L.Hkv), dim3(1024), 0, st, umask, nv, L.v0, u_cap, grp_idx, grp_mask,
                     grp_cnt);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

int run_visual_subset(const Layer& L, const int* kv_idx, const int* budget, int b_cap, int* vis_idx, int* vis_cnt,
                      hipStream_t st) {
  hipLaunchKernelGGL(visual_subset_kernel, dim3(L.B * L.Hq), dim3(256), 0, st, kv_idx, budget, L.bph, L.Hq, b_cap, L.v0, L.v1,
                     vis_idx, vis_cnt);
  OMNI_LAUNCH_CHECK();
  return OMNI_OK;
}

}  // namespace omni
