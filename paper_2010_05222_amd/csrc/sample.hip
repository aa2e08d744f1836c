// Positive-preserving negative sampling and label remap on one class shard
// (Partial FC, Sec. 3.3.1-3.3.2, Eq. local_sampling).
//
// S = P  union  {the n_neg = max(b - |P|, 0) non-positive classes with the
// smallest 64-bit Philox keys, ties to the lower class id}, sorted ascending,
// then labels_mapped = searchsorted(S, y - a).
//
// The keys are uniform, so the threshold (the n_neg-th smallest key) is known
// beforehand to within a few standard deviations, and one pass over the keys
// settles every class outside that window:
//   k_keys     positives of a group of classes (from the labels, in LDS), its
//              keys, and per class: surely in S (a positive, or a key below
//              the window), surely not (above), or a candidate, whose key is
//              written out;
//   k_resolve_write  the exact threshold among the candidates (by each
//              workgroup for itself), each group's place in S, S in class
//              order, and the labels' places in it.
// A shard of at most four groups does both in one launch (k_sample_one), and one with
// more than kMergeGroups groups finds the threshold once (k_resolve) before
// k_write.  If the count below the window or up to its end turns out wrong, the
// threshold is found over all keys, recomputed: 2.6 ms per million classes, and
// the same result.  That is 6e-7 of draws, but 2e-6 with a budget of 100 classes,
// 8e-6 with 10 and 5e-5 with one; and where only a few classes are left out, 2e-6
// with 100 of them, 4e-5 with 10 and 5e-4 with two.  When the budget is the whole
// shard nothing is drawn (k_take_all).  No host synchronisation, and no state
// that has to be cleared first.
//
// This replaces ten launches (clear, mark, plan, key digits and histogram, top
// digit, collect, refine, scan, write, remap), whose time was mostly that of
// empty launches: 10 K classes 55 -> 13 us, 100 K 46 -> 16 us, 2M 50 -> 23 us, 8M 76 -> 51 us.
#include <math.h>

#include "pfc_internal.h"

namespace pfc {
namespace {

// Philox4x64-10 (Salmon et al., SC'11): multipliers and Weyl key increments
// of the 4x64 variant.
constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kPhiloxW1 = 0xBB67AE8584CAA73Bull;

// N consecutive blocks from counter c0 on, their words in order.  The rounds are
// a loop over all blocks at once (independent chains) and not unrolled: a
// round of four blocks is about 1 KB of code, and on the small shards, where a
// kernel runs once from a cold instruction cache, ten times that cost more
// than the arithmetic.
template <int N>
__device__ __forceinline__ void philox4x64_10(uint64_t c0, uint64_t seed, uint64_t* out) {
  uint64_t x[N][4];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    x[i][0] = c0 + i;
    x[i][1] = x[i][2] = x[i][3] = 0;
  }
  uint64_t k0 = seed, k1 = 0;
#pragma unroll 1
  for (int r = 0; r < 10; ++r) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint64_t hi0 = __umul64hi(kPhiloxM0, x[i][0]);
      const uint64_t lo0 = kPhiloxM0 * x[i][0];
      const uint64_t hi1 = __umul64hi(kPhiloxM1, x[i][2]);
      const uint64_t lo1 = kPhiloxM1 * x[i][2];
      x[i][0] = hi1 ^ x[i][1] ^ k0;
      x[i][1] = lo1;
      x[i][2] = hi0 ^ x[i][3] ^ k1;
      x[i][3] = lo0;
    }
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) out[4 * i + e] = x[i][e];
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}

// Inclusive prefix sum over the wave by lane moves: shifts by 1, 2, 4, 8 inside
// each row of 16, then the last lanes of rows 0 and 2 into rows 1 and 3, and
// lane 31 into the upper half.  (Through __shfl, each step is an LDS round trip.)
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v = dpp_add<0x111, 0xF>(v);
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);
  return dpp_add<0x143, 0xC>(v);
}

// Exclusive prefix sum of `v` over the workgroup of kWaves waves (at most 16);
// `total` receives its sum.
template <int kWaves>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* smem, uint32_t* total) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t incl = wave_scan(v);
  if (lane_id() == 63) smem[wave] = incl;
  __syncthreads();
  const uint32_t sums = wave_scan(lane_id() < kWaves ? smem[lane_id()] : 0u);
  __syncthreads();
  *total = (uint32_t)__builtin_amdgcn_readlane((int)sums, kWaves - 1);
  const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)sums, wave - 1) : 0u;
  return before + incl - v;
}

// Three of them at once (v[i] becomes its exclusive prefix).
template <int kWaves>
__device__ __forceinline__ void block_scan3(uint32_t (&v)[3], uint32_t (*smem)[kWaves],
                                            uint32_t (&total)[3]) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t incl[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    incl[i] = wave_scan(v[i]);
    if (lane_id() == 63) smem[i][wave] = incl[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint32_t sums = wave_scan(lane_id() < kWaves ? smem[i][lane_id()] : 0u);
    total[i] = (uint32_t)__builtin_amdgcn_readlane((int)sums, kWaves - 1);
    const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)sums, wave - 1) : 0u;
    v[i] = before + incl[i] - v[i];
  }
  __syncthreads();
}

// Find the bin holding the k-th (1-based) element of an LDS histogram of kBins
// bins (two per thread of 1,024).  Returns through shared out[0] = bin, out[1] = count
// before the bin, out[2] = count of the bin (the last bin and zero counts if
// the histogram holds fewer than k).
constexpr int kBins = 2048;
__device__ __forceinline__ void find_kth_bin(const uint32_t* hist, int64_t k, uint32_t* smem,
                                             int64_t* out) {
  if (threadIdx.x == 0) {   // ordered before the writes below by the scan's barriers
    out[0] = kBins - 1;
    out[1] = 0;
    out[2] = 0;
  }
  const int b = 2 * threadIdx.x;
  const uint2 h = *reinterpret_cast<const uint2*>(hist + b);
  uint32_t total;
  const int64_t before = block_scan<16>(h.x + h.y, smem, &total);
  if (before < k && k <= before + h.x + h.y) {
    const bool second = before + h.x < k;
    out[0] = b + second;
    out[1] = before + (second ? h.x : 0u);
    out[2] = second ? h.y : h.x;
  }
  __syncthreads();
}

// ------------------------------------------------------------ group of classes

// Keys of the sixteen classes c0 .. c0 + 15 (c0 a multiple of 16) in the words
// of their Philox blocks: key q is that of class c0 + q - o, o = (a + c0) % 4
// (the shard may start inside a block; classes outside are neighbours').
__device__ __forceinline__ void keys16(uint64_t seed, int64_t a, int64_t c0, uint64_t (&keys)[20]) {
  const int64_t g = a + c0;
  philox4x64_10<4>((uint64_t)(g >> 2), seed, keys);
  if (g & 3) philox4x64_10<1>((uint64_t)(g >> 2) + 4, seed, keys + 16);
}

// f(i, key) for the classes i of `take`, c0 + i, in order.
template <typename F>
__device__ __forceinline__ void for_taken(uint32_t take, int o, const uint64_t (&keys)[20],
                                          F&& f) {
#pragma unroll
  for (int q = 0; q < 20; ++q) {
    if (q >= 16 && o == 0) break;
    if (q >= o && ((take >> (q - o)) & 1u)) f(q - o, keys[q]);
  }
}

__device__ __forceinline__ uint32_t live16(int64_t c0, int64_t C) {
  return c0 >= C ? 0u : C - c0 >= kPerThread ? 0xFFFFu : (1u << (C - c0)) - 1u;
}

// f(k, labels[k]) for every label, once across the workgroup, U loads in
// flight per thread (eight of 256 threads: one at a time they were 6 of k_keys'
// 16 us at B = 4096; fewer of 1,024 threads, whose code is then shorter);
// `before` runs once the first ones are requested.
template <int U, typename Before, typename F>
__device__ __forceinline__ void for_labels(const int64_t* labels, int64_t B, Before&& before,
                                           F&& f) {
  uint64_t y[U];
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + (int64_t)u * blockDim.x;
      y[u] = k < B ? (uint64_t)labels[k] : 0;
    }
  };
  load(threadIdx.x);
  before();
#pragma unroll 1
  for (int64_t k0 = threadIdx.x; k0 < B; k0 += (int64_t)U * blockDim.x) {
    if (k0 != threadIdx.x) load(k0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + (int64_t)u * blockDim.x;
      if (k < B) f(k, y[u]);
    }
  }
}

// The positives among the classes [c_lo, c_lo + n) (n a multiple of 32), as a
// bitmap in LDS.  Ends with a barrier.
template <int U>
__device__ __forceinline__ void mark_positives(const int64_t* labels, int64_t B, int64_t a,
                                               int64_t c_lo, int n, uint32_t* bits) {
  for_labels<U>(
      labels, B,
      [&] {
        for (int i = threadIdx.x; i < n / 32; i += blockDim.x) bits[i] = 0u;
        __syncthreads();
      },
      [&](int64_t, uint64_t y) {
        // Unsigned: a label before the range wraps far past its end.
        const uint64_t c = y - (uint64_t)(a + c_lo);
        if (c < (uint64_t)n) atomicOr(&bits[c >> 5], 1u << (c & 31));
      });
  __syncthreads();
}

// A thread's sixteen classes: masks of the positives, of the classes surely in
// S and of the candidates.
struct Masks {
  uint32_t pos, sure, in;
};

// Those of the classes from c0 on, and their keys; `bits` is the bitmap from
// class c0 - 16 t on.
__device__ __forceinline__ Masks draw16(const uint32_t* bits, int t, int64_t c0, int64_t C,
                                        int64_t a, uint64_t seed, uint32_t lo, uint32_t hi,
                                        uint64_t (&keys)[20]) {
  const uint32_t live = live16(c0, C);
  uint32_t below = 0, in = 0;
  if (live) {
    keys16(seed, a, c0, keys);
    const int o = (int)((a + c0) & 3);
    for_taken(live, o, keys, [&](int i, uint64_t key) {
      const uint32_t top = (uint32_t)(key >> 32);
      below |= (uint32_t)(top < lo) << i;
      in |= (uint32_t)(top >= lo && top <= hi) << i;
    });
  }
  const uint32_t pos = (bits[t >> 1] >> (16 * (t & 1))) & live;
  return Masks{pos, below | pos, in & ~pos};
}

// One workgroup per run of groups.  The candidates' keys go to the group's own
// part of cand_key in class order; masks keeps each thread's three masks and
// (top 16 bits) its first candidate's place.  Bound by the generator (about
// 300 instructions per four keys, a third of them multiplications at a quarter
// of the rate) on a large shard, by its latency on a small one: groups of 4,096
// classes spread it over four times the CUs that groups of 16,384 do (100 K
// classes: 6.9 against 11.6 us).
__global__ void __launch_bounds__(kGroupThreads) k_keys(
    const int64_t* labels, int64_t B, int64_t C, int64_t a, uint64_t seed, uint32_t lo,
    uint32_t hi, int64_t n_groups, int run, uint64_t* masks, uint64_t* cand_key,
    uint32_t* grp_sure, uint32_t* grp_cand) {
  __shared__ uint32_t bits[kGroupClasses / 32 * kRunMax];
  __shared__ uint32_t smem[kGroupThreads / 64];
  const int64_t g0 = (int64_t)blockIdx.x * run;
  const int n = (int)(n_groups - g0 < run ? n_groups - g0 : run);
  const int t = threadIdx.x;
  mark_positives<8>(labels, B, a, g0 * kGroupClasses, n * kGroupClasses, bits);
#pragma unroll 1
  for (int i = 0; i < n; ++i) {
    const int64_t g = g0 + i;
    const int64_t c0 = g * kGroupClasses + t * kPerThread;
    uint64_t keys[20];
    const Masks m = draw16(bits + kGroupClasses / 32 * i, t, c0, C, a, seed, lo, hi, keys);
    // Surely selected classes and candidates (at most 4,096 each) in one scan.
    uint32_t total, n_pos;
    const uint32_t pre = block_scan<kGroupThreads / 64>(
        (uint32_t)__popc(m.sure) | ((uint32_t)__popc(m.in) << 16), smem, &total) >> 16;
    block_scan<kGroupThreads / 64>((uint32_t)__popc(m.pos), smem, &n_pos);
    if (t == 0) {
      grp_sure[g] = (total & 0xFFFFu) | (n_pos << 16);
      grp_cand[g] = total >> 16;
    }
    masks[g * kGroupThreads + t] = (uint64_t)m.pos | ((uint64_t)m.sure << 16) |
                                   ((uint64_t)m.in << 32) | ((uint64_t)pre << 48);
    uint64_t* out = cand_key + g * kGroupClasses + pre;
    for_taken(m.in, (int)((a + c0) & 3), keys, [&](int, uint64_t key) { *out++ = key; });
  }
}

// ------------------------------------------------------------------ threshold
//
// All kernels from here on have 1,024 threads.

constexpr int kThreads = 1024;
constexpr int kSpan = kThreads * kPerThread;   // classes of a workgroup: four groups
constexpr int kSpanGroups = kSpan / kGroupClasses;
constexpr int kLastKeys = 512;    // keys ranked directly
constexpr int kListMax = 8192;    // candidates held in LDS

// A class is taken if its key is below `key`, or equal to it and (in class
// order) among the first `ties` such; `all_ties`: every such key is.
struct Threshold {
  uint64_t key;
  int64_t ties;
  bool all_ties;
  __device__ bool below(uint64_t k) const { return k < key || (all_ties && k == key); }
  __device__ bool tie(uint64_t k) const { return !all_ties && k == key; }
};

struct ResolveLds {
  __attribute__((aligned(8))) uint32_t hist[kBins];
  uint64_t last[kLastKeys];
  uint32_t scan[kThreads / 64];
  int64_t found[3];
  Threshold th;
  uint32_t n_last;
};

// The k-th (1-based) smallest of the keys that each(f) calls f on, once each
// across the workgroup; only those in [from, to] count.  The range is cut into
// bins until the one that holds the k-th key can be ranked directly, or holds
// one key value only.
template <typename Each>
__device__ __forceinline__ Threshold kth_key(Each&& each, int64_t k, uint64_t from, uint64_t to,
                                             ResolveLds& L) {
  const int t = threadIdx.x;
#pragma unroll 1
  for (;;) {
    const int width = 64 - __clzll((long long)(to - from));
    const int shift = width > 11 ? width - 11 : 0;
    *reinterpret_cast<uint2*>(L.hist + 2 * t) = make_uint2(0u, 0u);
    if (t == 0) L.n_last = 0;
    __syncthreads();
    each([&](uint64_t key) {
      if (key >= from && key <= to) atomicAdd(&L.hist[(key - from) >> shift], 1u);
    });
    __syncthreads();
    find_kth_bin(L.hist, k, L.scan, L.found);
    from += (uint64_t)L.found[0] << shift;
    k -= L.found[1];
    const int64_t n = L.found[2];
    // The bin's end, not past the range's: from there on it may not be a number.
    const uint64_t span = (1ull << shift) - 1ull;
    to = to - from < span ? to : from + span;
    if (shift == 0) return Threshold{from, k, k == n};
    if (n <= kLastKeys) {
      each([&](uint64_t key) {
        if (key < from || key > to) return;
        const uint32_t i = atomicAdd(&L.n_last, 1u);
        if (i < kLastKeys) L.last[i] = key;   // n of them: what the bin counted
      });
      __syncthreads();
      if (t < (int)n) {
        const uint64_t key = L.last[t];
        int64_t less = 0, equal = 0;
#pragma unroll 1
        for (int i = 0; i < (int)n; ++i) {
          less += L.last[i] < key;
          equal += L.last[i] == key;
        }
        if (less < k && k <= less + equal) L.th = Threshold{key, k - less, k == less + equal};
      }
      __syncthreads();
      return L.th;
    }
    __syncthreads();   // found is read before the next pass rewrites it
  }
}

// The threshold over all keys of the shard's non-positives, recomputed.  Inlined:
// as a function it saved its callers' registers on the stack, and a kernel with
// a stack makes the runtime allocate device memory at its first launch.
__device__ __forceinline__ Threshold kth_of_all(const uint64_t* masks, int64_t C, int64_t a,
                                                uint64_t seed, int64_t n_neg, ResolveLds& L) {
  return kth_key(
      [&](auto&& f) {
        for (int64_t v = threadIdx.x; v * kPerThread < C; v += kThreads) {
          uint64_t keys[20];
          keys16(seed, a, v * kPerThread, keys);
          for_taken(live16(v * kPerThread, C) & ~(uint32_t)(masks[v] & 0xFFFFu), (int)(a & 3),
                    keys, [&](int, uint64_t key) { f(key); });
        }
      },
      n_neg, 0, ~0ull, L);
}

// From the shard's |P|, its non-positives below the window and its candidates:
// the rank of the threshold among the candidates, or -1 when the window missed
// it.  (With n_neg = 0 nothing is below the window either, since one that
// starts above 0 leaves n_neg > 0: rank 0, no candidate.)
__device__ __forceinline__ int64_t candidate_rank(int64_t budget, int64_t pos, int64_t below,
                                                  int64_t cand, int64_t* n_neg) {
  *n_neg = budget > pos ? budget - pos : 0;
  const int64_t k = *n_neg - below;
  return k < 0 || k > cand ? -1 : k;
}

// Masks of a thread's classes in S and of its ties, with the threshold over
// all keys.
__device__ __attribute__((noinline)) uint2 settle_all(uint32_t pos, int64_t c0, int64_t C,
                                                      int64_t a, uint64_t seed, Threshold th) {
  const uint32_t take = live16(c0, C) & ~pos;
  uint32_t sel = pos, tie = 0;
  if (take) {
    uint64_t keys[20];
    keys16(seed, a, c0, keys);
    for_taken(take, (int)((a + c0) & 3), keys, [&](int i, uint64_t key) {
      sel |= (uint32_t)th.below(key) << i;
      tie |= (uint32_t)th.tie(key) << i;
    });
  }
  return make_uint2(sel, tie);
}

// The same from the thread's packed masks: of its candidates, whose keys start
// at list, those that the threshold takes join the sure ones; no candidate
// with k = 0, and all keys decide with k < 0.
__device__ __forceinline__ uint2 settle(uint64_t m, const uint64_t* list, int64_t k,
                                        const Threshold& th, int64_t c0, int64_t C, int64_t a,
                                        uint64_t seed) {
  if (k < 0) return settle_all((uint32_t)(m & 0xFFFFu), c0, C, a, seed, th);
  uint32_t sel = (uint32_t)(m >> 16) & 0xFFFFu, tie = 0;
  if (k > 0) {
    const uint64_t* next = list + (m >> 48);
    for (uint32_t rest = (uint32_t)(m >> 32) & 0xFFFFu; rest; rest &= rest - 1) {
      const uint64_t key = *next++;
      if (th.below(key)) sel |= rest & (0u - rest);
      if (th.tie(key)) tie |= rest & (0u - rest);
    }
  }
  return make_uint2(sel, tie);
}

// -------------------------------------------------------------------- output

// A workgroup's span of classes in S, sixteen per thread from c0 on: `st.x` for
// sure and, of `st.y`, the first that th.ties leaves after `tie_before`.  The
// ids go to active[out ..), and where[t] keeps the thread's mask in the low
// half, its first place relative to the span's in the high half.
__device__ __forceinline__ void write_span(uint2 st, const Threshold& th, int64_t out,
                                           int64_t tie_before, int64_t c0, int64_t cap,
                                           int32_t* active, uint32_t* smem, uint32_t* where) {
  uint32_t sel = st.x, total;
  if (!th.all_ties && th.ties) {
    int64_t before = tie_before + block_scan<16>((uint32_t)__popc(st.y), smem, &total);
    for (uint32_t rest = st.y; rest; rest &= rest - 1)
      if (before++ < th.ties) sel |= rest & (0u - rest);
  }
  const uint32_t pre = block_scan<16>((uint32_t)__popc(sel), smem, &total);
  where[threadIdx.x] = sel | (pre << 16);
  int64_t o = out + pre;
  for (uint32_t rest = sel; rest; rest &= rest - 1, ++o)
    if (o < cap) active[o] = (int32_t)(c0 + __ffs(rest) - 1);
}

// Places of the labels in n spans of classes from class c_lo on, which start at
// out[0 .. n) in S; the first workgroup also marks the labels outside the
// shard.  Every in-shard label is a positive, which S always holds; one that
// it did not hold would be mapped to -1 (unowned), never to another class's
// place or past |S|.
__device__ __forceinline__ void map_labels(const int64_t* labels, int64_t B, int64_t C, int64_t a,
                                           int64_t c_lo, int n, const uint32_t* out,
                                           const uint32_t* where, int64_t cap,
                                           int32_t* labels_mapped) {
  for_labels<1>(labels, B, [] { __syncthreads(); }, [&](int64_t k, uint64_t label) {
    const uint64_t y = label - (uint64_t)a;
    if (y >= (uint64_t)C) {
      if (c_lo == 0) labels_mapped[k] = -1;
      return;
    }
    const uint64_t c = y - (uint64_t)c_lo;
    if (c >= (uint64_t)n * kSpan) return;
    const uint32_t p = where[c / kPerThread];
    const int i = (int)(c % kPerThread);
    const int64_t o = (int64_t)out[c / kSpan] + (p >> 16) + __popc(p & ((1u << i) - 1u));
    labels_mapped[k] = ((p >> i) & 1u) && o < cap ? (int32_t)o : -1;
  });
}

// Of `tie` ties, those taken when `before` precede them.
__device__ __forceinline__ uint32_t taken(const Threshold& th, int64_t before, uint32_t tie) {
  const int64_t left = th.ties - before;
  return left <= 0 ? 0u : left < (int64_t)tie ? (uint32_t)left : tie;
}

// |S| <= cap by construction; the clamp keeps every later index in bounds.
__device__ __forceinline__ int32_t clamp_count(uint64_t n, int64_t cap) {
  return (int32_t)(n < (uint64_t)cap ? n : (uint64_t)cap);
}

// A shard of at most one span: everything in one workgroup.
__global__ void __launch_bounds__(kThreads) k_sample_one(
    const int64_t* labels, int64_t B, int64_t C, int64_t a, uint64_t seed, int64_t budget,
    uint32_t lo, uint32_t hi, int64_t cap, uint64_t* masks, int32_t* active, int32_t* n_active,
    int32_t* labels_mapped) {
  __shared__ ResolveLds L;
  __shared__ uint32_t bits[kSpan / 32], where[kThreads];
  __shared__ uint64_t list[kSpan];
  __shared__ uint32_t out;
  const int t = threadIdx.x;
  const int64_t c0 = t * kPerThread;
  mark_positives<2>(labels, B, a, 0, kSpan, bits);
  uint64_t m;
  uint32_t total, n_pos;
  {
    uint64_t keys[20];
    const Masks d = draw16(bits, t, c0, C, a, seed, lo, hi, keys);
    const uint32_t pre = block_scan<16>((uint32_t)__popc(d.sure) | ((uint32_t)__popc(d.in) << 16),
                                        L.scan, &total) >> 16;
    block_scan<16>((uint32_t)__popc(d.pos), L.scan, &n_pos);
    uint64_t* next = list + pre;
    for_taken(d.in, (int)(a & 3), keys, [&](int, uint64_t key) { *next++ = key; });
    m = (uint64_t)d.pos | ((uint64_t)d.sure << 16) | ((uint64_t)d.in << 32) | ((uint64_t)pre << 48);
  }
  int64_t n_neg;
  const int64_t k = candidate_rank(budget, n_pos, (int64_t)(total & 0xFFFFu) - n_pos, total >> 16,
                                   &n_neg);
  Threshold th{0, 0, false};
  if (k > 0) {   // kth_key's first barrier completes the list
    th = kth_key(
        [&](auto&& f) {
          for (uint32_t i = t; i < total >> 16; i += kThreads) f(list[i]);
        },
        k, (uint64_t)lo << 32, ((uint64_t)hi << 32) | 0xFFFFFFFFu, L);
  } else if (k < 0) {
    masks[t] = m;
    __syncthreads();
    th = kth_of_all(masks, C, a, seed, n_neg, L);
  }
  if (t == 0) {
    out = 0;
    *n_active = clamp_count((uint64_t)n_pos + (uint64_t)n_neg, cap);
  }
  write_span(settle(m, list, k, th, c0, C, a, seed), th, 0, 0, c0, cap, active, L.scan, where);
  map_labels(labels, B, C, a, 0, 1, &out, where, cap, labels_mapped);
}

// Calls f(group, i, key) on candidate i of the groups, once across the
// workgroup, 1 << lane_bits threads to a group so that they read its list in
// one piece (few lanes per group read short pieces of many lists at a time, a
// cache line each), eight groups' loads in flight per thread.  count(g) is the
// group's number of candidates.
template <typename Count, typename F>
__device__ __forceinline__ void for_candidates(const uint64_t* cand_key, int64_t n_groups,
                                               int lane_bits, Count&& count, F&& f) {
  constexpr int U = 8;
  const uint32_t lanes = 1u << lane_bits, sub = threadIdx.x & (lanes - 1);
  const int64_t step = kThreads >> lane_bits;
#pragma unroll 1
  for (int64_t g0 = threadIdx.x >> lane_bits; g0 < n_groups; g0 += U * step) {
    uint32_t n[U];
    uint64_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) n[u] = g0 + u * step < n_groups ? count(g0 + u * step) : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = sub < n[u] ? cand_key[(g0 + u * step) * kGroupClasses + sub] : 0;
    bool more = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (sub < n[u]) f(g0 + u * step, sub, v[u]);
      more |= sub + lanes < n[u];
    }
    if (more) {   // longer lists than expected
#pragma unroll 1
      for (int64_t g = g0; g < n_groups && g < g0 + U * step; g += step)
        for (uint32_t i = sub + lanes; i < count(g); i += lanes)
          f(g, i, cand_key[g * kGroupClasses + i]);
    }
  }
}

// At most kMergeGroups groups: each workgroup gathers all candidates into LDS
// (1 << lane_bits threads per group), resolves the threshold, counts all
// groups (1 << count_bits lanes of a wave each), and writes its own span.
__global__ void __launch_bounds__(kThreads) k_resolve_write(
    SampleWs w, const int64_t* labels, int64_t B, int64_t C, int64_t a, uint64_t seed,
    int n_groups, int lane_bits, int count_bits, int64_t budget, uint32_t lo, uint32_t hi, int64_t cap,
    int32_t* active, int32_t* n_active, int32_t* labels_mapped) {
  __shared__ ResolveLds L;
  __shared__ uint64_t list[kListMax];
  __shared__ uint32_t where[kThreads];
  __shared__ uint32_t start[kMergeGroups + 1];   // of each group's candidates in the list
  __shared__ uint32_t cnt[2][kMergeGroups];
  __shared__ uint32_t scan3[3][16];
  __shared__ uint32_t out, tie_before;
  const int t = threadIdx.x;
  const int64_t c0 = ((int64_t)blockIdx.x * kThreads + t) * kPerThread;
  const int g_own = blockIdx.x * kSpanGroups;
  const bool own = c0 < (int64_t)n_groups * kGroupClasses;
  const uint64_t m = own ? w.masks[c0 / kPerThread] : 0;
  const uint32_t sure = t < n_groups ? w.grp_sure[t] : 0u;
  const uint32_t n_cand = t < n_groups ? w.grp_cand[t] : 0u;
  uint32_t v[3] = {sure >> 16, (sure & 0xFFFFu) - (sure >> 16), n_cand}, sum[3];
  block_scan3<16>(v, scan3, sum);
  const uint32_t pos = sum[0], below = sum[1], cand = sum[2];
  if (t < n_groups) start[t] = v[2];
  if (t == 0) start[n_groups] = cand;
  __syncthreads();
  int64_t n_neg;
  const int64_t k = candidate_rank(budget, pos, below, cand, &n_neg);
  const bool fits = cand <= (uint32_t)kListMax;
  auto from_memory = [&](auto&& f) {
    for_candidates(w.cand_key, n_groups, lane_bits,
                   [&](int64_t g) { return start[g + 1] - start[g]; }, f);
  };
  Threshold th{0, 0, false};
  if (k > 0) {
    if (fits)
      from_memory([&](int64_t g, uint32_t i, uint64_t key) { list[start[g] + i] = key; });
    // kth_key's first barrier completes the list.
    th = kth_key(
        [&](auto&& f) {
          if (fits) {
            for (uint32_t i = t; i < cand; i += kThreads) f(list[i]);
          } else {
            from_memory([&](int64_t, uint32_t, uint64_t key) { f(key); });
          }
        },
        k, (uint64_t)lo << 32, ((uint64_t)hi << 32) | 0xFFFFFFFFu, L);
  } else if (k < 0) {
    th = kth_of_all(w.masks, C, a, seed, n_neg, L);
  }

  const int lanes = 1 << count_bits, sub = t & (lanes - 1);
  // Each group's classes in S and its ties: its lanes' votes, counted by all of
  // them (sums by lane moves, ten LDS round trips a group, took 5 us of 17 on
  // 245 groups).
  const uint64_t group_lanes = (lanes == 64 ? ~0ull : ((1ull << lanes) - 1ull) << (lane_id() & ~(lanes - 1)));
#pragma unroll 1
  for (int g = t >> count_bits; g < n_groups; g += kThreads >> count_bits) {
    uint32_t s = 0, e = 0;
    if (k > 0) {
      const uint32_t n = start[g + 1] - start[g];
      for (uint32_t i = sub; i < n; i += lanes) {
        const uint64_t key =
            fits ? list[start[g] + i] : w.cand_key[(int64_t)g * kGroupClasses + i];
        s += __popcll(__ballot(th.below(key)) & group_lanes);
        e += __popcll(__ballot(th.tie(key)) & group_lanes);
      }
    } else if (k < 0) {
      for (int v = sub; v < kGroupThreads; v += lanes) {
        const int64_t at = (int64_t)g * kGroupThreads + v;
        const uint2 st = settle_all((uint32_t)(w.masks[at] & 0xFFFFu), at * kPerThread, C, a,
                                    seed, th);
        s += __popc(st.x);
        e += __popc(st.y);
      }
      for (int off = 1; off < lanes; off <<= 1) {
        s += __shfl_xor(s, off, 64);
        e += __shfl_xor(e, off, 64);
      }
    }
    if (sub == 0) {   // in every vote of the group
      cnt[0][g] = s;
      cnt[1][g] = e;
    }
  }
  __syncthreads();
  uint32_t s = t < n_groups ? cnt[0][t] + (k >= 0 ? sure & 0xFFFFu : 0u) : 0u;
  uint32_t tb = 0, total;
  if (!th.all_ties && th.ties) {
    const uint32_t e = t < n_groups ? cnt[1][t] : 0u;
    tb = block_scan<16>(e, L.scan, &total);
    s += taken(th, tb, e);
  }
  const uint32_t ob = block_scan<16>(s, L.scan, &total);
  if (t == g_own) {
    out = ob;
    tie_before = tb;
  }
  if (g_own == 0 && t == 0) *n_active = clamp_count(total, cap);
  __syncthreads();
  const uint64_t* keys = w.cand_key + c0 / kGroupClasses * kGroupClasses;
  const uint2 st = own ? settle(m, keys, k, th, c0, C, a, seed) : make_uint2(0u, 0u);
  write_span(st, th, out, tie_before, c0, cap, active, L.scan, where);
  map_labels(labels, B, C, a, (int64_t)blockIdx.x * kSpan, 1, &out, where, cap, labels_mapped);
}

// More groups: the threshold, then each group's classes in S and ties, turned
// into offsets.  One workgroup, 1 << lane_bits <= 64 lanes of a wave per group.
// Bound by memory latency: the candidates of up to kHeldGroups groups are read
// once, into LDS, if they fit, and counted there by votes (8M classes, B = 1024:
// 22 us; 38 with two passes over memory for the threshold and a third that
// summed each group's counts by lane moves).  LDS holds the upper
// 32 bits of a candidate's place in the window; where they do not tell the
// threshold from a neighbour (4e-6 of draws), and for longer lists, every pass
// reads memory, eight groups' loads in flight per thread.
constexpr int kHeldGroups = 8 * kThreads;
constexpr int kHeldPer = kHeldGroups / kThreads;
constexpr int kHeldMax = 28672;
__global__ void __launch_bounds__(kThreads) k_resolve(SampleWs w, int64_t n_groups, int lane_bits,
                                                      int64_t C, int64_t a, uint64_t seed,
                                                      int64_t budget, uint32_t lo, uint32_t hi,
                                                      int64_t cap, int32_t* n_active) {
  __shared__ ResolveLds L;
  __shared__ uint32_t list[kHeldMax];
  __shared__ uint16_t start[kHeldGroups + 1];   // of each group's candidates in the list
  __shared__ uint16_t counts[kHeldGroups];      // of the held candidates that are taken
  __shared__ uint32_t scan3[3][16];
  const int t = threadIdx.x;
  const int lanes = 1 << lane_bits, sub = t & (lanes - 1);
  const uint64_t group_lanes =
      lanes == 64 ? ~0ull : ((1ull << lanes) - 1ull) << (lane_id() & ~(lanes - 1));
  const uint64_t from = (uint64_t)lo << 32, to = ((uint64_t)hi << 32) | 0xFFFFFFFFu;
  // Eight consecutive groups per thread and pass.
  uint32_t v[3] = {0u, 0u, 0u}, sum[3], nc[kHeldPer];
#pragma unroll 1
  for (int64_t base = kHeldPer * t; base < n_groups; base += kHeldGroups) {
    uint32_t sure[kHeldPer];
#pragma unroll
    for (int i = 0; i < kHeldPer; ++i) {
      sure[i] = base + i < n_groups ? w.grp_sure[base + i] : 0u;
      nc[i] = base + i < n_groups ? w.grp_cand[base + i] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kHeldPer; ++i) {
      v[0] += sure[i] >> 16;
      v[1] += (sure[i] & 0xFFFFu) - (sure[i] >> 16);
      v[2] += nc[i];
    }
  }
  block_scan3<16>(v, scan3, sum);
  const uint32_t pos = sum[0], below = sum[1], cand = sum[2];
  int64_t n_neg;
  const int64_t k = candidate_rank(budget, pos, below, cand, &n_neg);
  bool held = k > 0 && n_groups <= kHeldGroups && cand <= (uint32_t)kHeldMax;
  Threshold th{0, 0, false};
  if (held) {
#pragma unroll
    for (int i = 0; i < kHeldPer; ++i) {
      if (kHeldPer * t + i >= n_groups) break;
      start[kHeldPer * t + i] = (uint16_t)v[2];
      v[2] += nc[i];
    }
    if (t == 0) start[n_groups] = (uint16_t)cand;
    __syncthreads();
    // The window is hi - lo + 1 <= 2^drop times 2^32 keys.
    const int drop = hi > lo ? 32 - __clz((int)(hi - lo)) : 0;
    for_candidates(w.cand_key, n_groups, lane_bits,
                   [&](int64_t g) { return (uint32_t)start[g + 1] - start[g]; },
                   [&](int64_t g, uint32_t i, uint64_t key) {
                     list[start[g] + i] = (uint32_t)((key - from) >> drop);
                   });
    // kth_key's first barrier completes the list.
    const Threshold at = kth_key(
        [&](auto&& f) {
          for (uint32_t i = t; i < cand; i += kThreads) f((uint64_t)list[i]);
        },
        k, 0, 0xFFFFFFFFull, L);
    held = at.all_ties;   // all candidates with these 32 bits are taken
    if (held) {
      th = Threshold{from + (((at.key + 1) << drop) - 1), at.ties, true};
#pragma unroll 1
      for (int g = t >> lane_bits; g < (int)n_groups; g += kThreads >> lane_bits) {
        const uint32_t first = start[g], n = start[g + 1] - first;
        uint32_t s = 0;
        for (uint32_t i = sub; i < n; i += lanes)
          s += __popcll(__ballot(list[first + i] <= (uint32_t)at.key) & group_lanes);
        if (sub == 0) counts[g] = (uint16_t)s;   // sub 0 is in every vote of the group
      }
    }
  }
  if (!held && k > 0) {
    th = kth_key(
        [&](auto&& f) {
          for_candidates(w.cand_key, n_groups, lane_bits, [&](int64_t g) { return w.grp_cand[g]; },
                         [&](int64_t, uint32_t, uint64_t key) { f(key); });
        },
        k, from, to, L);
    constexpr int U = 8;
    const int64_t step = kThreads >> lane_bits;
#pragma unroll 1
    for (int64_t g0 = t >> lane_bits; g0 < n_groups; g0 += U * step) {
      uint32_t n[U], s[U], e[U];
      uint64_t key[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t g = g0 + u * step;
        n[u] = g < n_groups ? w.grp_cand[g] : 0u;
        s[u] = g < n_groups ? w.grp_sure[g] & 0xFFFFu : 0u;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        key[u] = sub < n[u] ? w.cand_key[(g0 + u * step) * kGroupClasses + sub] : 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        s[u] += __popcll(__ballot(sub < n[u] && th.below(key[u])) & group_lanes);
        e[u] = __popcll(__ballot(sub < n[u] && th.tie(key[u])) & group_lanes);
#pragma unroll 1
        for (uint32_t i = sub + lanes; i < n[u]; i += lanes) {   // longer than expected
          const uint64_t more = w.cand_key[(g0 + u * step) * kGroupClasses + i];
          s[u] += __popcll(__ballot(th.below(more)) & group_lanes);
          e[u] += __popcll(__ballot(th.tie(more)) & group_lanes);
        }
        if (sub == 0 && g0 + u * step < n_groups) {
          w.grp_out[g0 + u * step] = s[u];
          w.grp_tie_off[g0 + u * step] = e[u];
        }
      }
    }
  } else if (!held) {
    if (k < 0) th = kth_of_all(w.masks, C, a, seed, n_neg, L);
#pragma unroll 1
    for (int64_t g = t >> lane_bits; g < n_groups; g += kThreads >> lane_bits) {
      uint32_t s = 0, e = 0;
      for (int u = sub; k < 0 && u < kGroupThreads; u += lanes) {
        const int64_t at = g * kGroupThreads + u;
        const uint2 st = settle_all((uint32_t)(w.masks[at] & 0xFFFFu), at * kPerThread, C, a,
                                    seed, th);
        s += __popc(st.x);
        e += __popc(st.y);
      }
      for (int off = 1; off < lanes; off <<= 1) {
        s += __shfl_xor(s, off, 64);
        e += __shfl_xor(e, off, 64);
      }
      if (sub == 0) {
        w.grp_out[g] = k < 0 ? s : w.grp_sure[g] & 0xFFFFu;
        w.grp_tie_off[g] = e;
      }
    }
  }
  __syncthreads();
  const bool part = !th.all_ties && th.ties;   // only some of the ties are taken
  uint64_t all_tie = 0, all_sel = 0;
#pragma unroll 1
  for (int64_t base = kHeldPer * t; base - kHeldPer * t < n_groups; base += kHeldGroups) {
    uint32_t s[kHeldPer], e[kHeldPer], s_all = 0, e_all = 0, total;
#pragma unroll
    for (int i = 0; i < kHeldPer; ++i) {
      const int64_t g = base + i;
      const bool in = g < n_groups;
      s[i] = !in ? 0u : held ? counts[g] + (w.grp_sure[g] & 0xFFFFu) : w.grp_out[g];
      e[i] = in && part ? w.grp_tie_off[g] : 0u;
      e_all += e[i];
    }
    if (part) {
      uint64_t tb = all_tie + block_scan<16>(e_all, L.scan, &total);
      all_tie += total;
#pragma unroll
      for (int i = 0; i < kHeldPer; ++i) {
        if (base + i < n_groups) w.grp_tie_off[base + i] = (uint32_t)tb;
        s[i] += taken(th, (int64_t)tb, e[i]);
        tb += e[i];
      }
    }
#pragma unroll
    for (int i = 0; i < kHeldPer; ++i) s_all += s[i];
    uint64_t ob = all_sel + block_scan<16>(s_all, L.scan, &total);
    all_sel += total;
#pragma unroll
    for (int i = 0; i < kHeldPer; ++i) {
      if (base + i < n_groups) w.grp_out[base + i] = (uint32_t)ob;
      ob += s[i];
    }
  }
  if (t == 0) {
    *w.state = SampleState{th.key, th.ties, k, th.all_ties};
    *n_active = clamp_count(all_sel, cap);
  }
}

// One workgroup per run of spans.
__global__ void __launch_bounds__(kThreads) k_write(
    SampleWs w, const int64_t* labels, int64_t B, int64_t C, int64_t a, uint64_t seed,
    int64_t n_groups, int run, int64_t cap, int32_t* active, int32_t* labels_mapped) {
  __shared__ uint32_t smem[kThreads / 64];
  __shared__ uint32_t where[kThreads * kSpanRunMax];
  __shared__ uint32_t out[kSpanRunMax];
  const int t = threadIdx.x;
  const int64_t s0 = (int64_t)blockIdx.x * run;
  const int64_t n_spans = ceil_div(n_groups, (int64_t)kSpanGroups);
  const int n = (int)(n_spans - s0 < run ? n_spans - s0 : run);
  const SampleState z = *w.state;
  const Threshold th{z.thresh, z.ties, z.all_ties};
  if (t < n) out[t] = w.grp_out[(s0 + t) * kSpanGroups];
#pragma unroll 1
  for (int i = 0; i < n; ++i) {
    const int64_t c0 = ((s0 + i) * kThreads + t) * kPerThread;
    const int64_t g = c0 / kGroupClasses;
    uint2 st = make_uint2(0u, 0u);
    if (g < n_groups)
      st = settle(w.masks[c0 / kPerThread], w.cand_key + g * kGroupClasses, z.rank, th, c0, C, a,
                  seed);
    write_span(st, th, w.grp_out[(s0 + i) * kSpanGroups], w.grp_tie_off[(s0 + i) * kSpanGroups],
               c0, cap, active, smem, where + kThreads * i);
  }
  map_labels(labels, B, C, a, s0 * kSpan, n, out, where, cap, labels_mapped);
}

// A budget of the whole shard: S is every class, whatever the keys.
__global__ void __launch_bounds__(256) k_take_all(const int64_t* labels, int64_t B, int64_t C,
                                                  int64_t a, int32_t* active, int32_t* n_active,
                                                  int32_t* labels_mapped) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  if (tid == 0) *n_active = (int32_t)C;
  for (int64_t i = tid; i < C; i += stride) active[i] = (int32_t)i;
  for (int64_t i = tid; i < B; i += stride) {
    const uint64_t y = (uint64_t)labels[i] - (uint64_t)a;
    labels_mapped[i] = y < (uint64_t)C ? (int32_t)y : -1;
  }
}

}  // namespace

// The window of the keys' top 32 bits that holds the threshold.  The number of
// keys below t is binomial with mean F = t C; the threshold lies where the
// non-positives among them are b - |P|, that is where F is between b - |P|
// (no positive below) and b (all of them), |P| <= min(B, C), give or take the
// deviation of F: five of its standard deviations at F = b, and four classes
// more.  (At the window's ends the deviation is another one, by a good part of
// itself where b or C - b is below a hundred: hence the rates of the misses above.)
void sample_window(int64_t B, int64_t C, int64_t budget, uint32_t* lo, uint32_t* hi) {
  const double b = (double)budget, c = (double)C, two32 = 4294967296.0;
  const double slack = 5.0 * sqrt(b * (1.0 - b / c)) + 4.0;
  const double from = (b - (double)(B < C ? B : C) - slack) / c * two32;
  const double to = (b + slack) / c * two32;
  *lo = from <= 0.0 ? 0u : (uint32_t)from;
  *hi = to >= two32 - 1.0 ? 0xFFFFFFFFu : (uint32_t)ceil(to);
}

hipError_t launch_sample(const int64_t* labels, int64_t B, int64_t C, int64_t a,
                         int64_t budget, uint64_t seed, int64_t n_groups, const SampleWs& w,
                         int32_t* active, int64_t cap, int32_t* n_active, int32_t* labels_mapped,
                         hipStream_t stream) {
  timing_start(0, stream);
  if (budget >= C) {
    const int64_t blocks = ceil_div(C > B ? C : B, 1024);
    hipLaunchKernelGGL(k_take_all, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(256), 0,
                       stream, labels, B, C, a, active, n_active, labels_mapped);
    timing_stop(0, stream);
    return hipGetLastError();
  }
  uint32_t lo, hi;
  sample_window(B, C, budget, &lo, &hi);
  if (C <= kSpan) {
    hipLaunchKernelGGL(k_sample_one, dim3(1), dim3(kThreads), 0, stream, labels, B, C, a, seed,
                       budget, lo, hi, cap, w.masks, active, n_active, labels_mapped);
    timing_stop(0, stream);
    return hipGetLastError();
  }
  // Each workgroup reads all labels: on very large shards it takes a run of
  // several groups, so that those reads stay below the generator's time.
  const int n = (int)n_groups;
  const int run = n / 2048 < 1 ? 1 : n / 2048 > kRunMax ? kRunMax : n / 2048;
  hipLaunchKernelGGL(k_keys, dim3((unsigned)ceil_div(n, run)), dim3(kGroupThreads), 0, stream,
                     labels, B, C, a, seed, lo, hi, n_groups, run, w.masks, w.cand_key, w.grp_sure,
                     w.grp_cand);
  // Threads that read a group's candidates: about as many as it has; at most a
  // wave where their counts are summed by lane moves.
  const double per_group = ((double)hi - (double)lo) / 4294967296.0 * kGroupClasses;
  int lane_bits = 0;
  while (lane_bits < 10 && (double)(1 << lane_bits) < per_group) ++lane_bits;
  const int count_bits = lane_bits < 6 ? lane_bits : 6;
  const int n_spans = (int)ceil_div(n, kSpanGroups);
  if (n <= kMergeGroups) {
    hipLaunchKernelGGL(k_resolve_write, dim3((unsigned)n_spans), dim3(kThreads), 0, stream, w,
                       labels, B, C, a, seed, n, lane_bits, count_bits, budget, lo, hi, cap, active,
                       n_active, labels_mapped);
  } else {
    const int span_run = n_spans / 512 < 1             ? 1
                         : n_spans / 512 > kSpanRunMax ? kSpanRunMax
                                                       : n_spans / 512;
    hipLaunchKernelGGL(k_resolve, dim3(1), dim3(kThreads), 0, stream, w, n_groups, count_bits, C,
                       a, seed, budget, lo, hi, cap, n_active);
    hipLaunchKernelGGL(k_write, dim3((unsigned)ceil_div(n_spans, span_run)), dim3(kThreads), 0,
                       stream, w, labels, B, C, a, seed, n_groups, span_run, cap, active,
                       labels_mapped);
  }
  timing_stop(0, stream);
  return hipGetLastError();
}

}  // namespace pfc
