// Load-balancing simulation for gfx950 (MI355X): host entry points and kernels.
// See lbs.h for what is simulated and for the contract of every call.
//
// A workgroup (256 threads, four wavefronts) runs one trial at a time and a share of
// the call's trials in turn.  Nothing here is a contraction or a stream over HBM: the
// work is integer ALU, cross-lane traffic and LDS, the outputs are two words per trial.
//
// A draw is one SplitMix64 output (a handful of 64-bit integer operations) and the
// inverse of the cumulative histogram at the index it selects.  The histogram sits in
// LDS, and so does a guide table made when the dataset is created: for every range
// the draws can come from (the whole dataset, each stratum) and every value (cell) of the
// draw's upper 11 (whole dataset) or 9 (stratum) bits.  Where the draws of a cell select one length, or two
// neighbouring ones, its entry says the first of them and the exact draw from which on it is the second: one LDS
// read and one addition give the length, with no search and no look at the histogram.  The other cells (flagged)
// hold the interval of lengths that they can select, which is searched.
//   NONE / STRATIFIED : a thread owns whole GPUs; local_batch draws, one sum each.
//   LOCAL_*           : (k_lbs_bins, node sizes and quotas that fit) a wavefront owns a node; its strata, which
//                       are disjoint ranges of lengths and take whole rows of the sorted pool, are packed into
//                       bins of 64 lanes, two bins to a register as 16-bit halves, and sorted there;
//                       (k_lbs_local, everything else) a wavefront owns a node.  Its lanes draw the node's pool into
//                       registers (entry i of the pool in register i / 64 of lane
//                       i % 64, padded to a multiple of 64 with a sentinel above every
//                       length) and sort it there with a bitonic network: a
//                       compare-exchange at distance < 64 is a cross-lane exchange, one
//                       at distance >= 64 pairs two registers of the same lane.  For a
//                       node of 1, 2, 4, ... 32 GPUs each GPU's column of the sorted pool
//                       is then summed across lanes; else the pool goes to LDS once, where
//                       each GPU's column is added up in raster or snake order.
//   GLOBAL            : lengths are small integers, so the trial's pool of
//                       n_gpus * local_batch draws is sorted by counting: an LDS
//                       histogram and a block-wide running sum give every length its
//                       range of sorted positions, which it spreads over the GPUs
//                       (position q goes to GPU q % n_gpus) through a difference array.
// Per-trial minimum and maximum are combined with shuffles and LDS; the two sums
// over trials are kept per workgroup and added up with 64-bit integer atomics at its
// end (integer addition is associative, so the result does not depend on the order).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "lbs.h"

namespace lbs {
// guide tables: indexed by a draw's upper 11 bits for the whole dataset, by its upper 9 bits for a stratum
constexpr uint32_t kWholeGuideBits = 11, kWholeGuideSize = 1u << kWholeGuideBits;
constexpr uint32_t kGuideBits = 9, kGuideSize = 1u << kGuideBits;
}

struct lbs_dataset {
  int device = -1;
  uint32_t max_len = 0, n_strata = 0;
  std::vector<uint32_t> cum, stratum_end;
  uint32_t* d_cum = nullptr;
  uint32_t n_cus = 1;           // compute units of the device
  bool flagged = false;         // some guide entry has to be searched
  uint32_t* d_guide = nullptr;  // the whole dataset's table (kWholeGuideSize entries), then one of kGuideSize per stratum
};

namespace lbs {
namespace {

constexpr uint32_t kBlock = 256, kWaves = 4;
constexpr uint32_t kMaxSpreadGpus = 8192;  // k_lbs_global keeps one LDS word per GPU up to here
// workgroups launched per compute unit (at most 8 are resident at a time): many short rounds, handed out as slots
// free up, balance better than few long ones (measured: 16 -> 6.4 ms, 32 -> 5.9, 64 -> 5.8, 128 -> 5.7 for the five
// methods at once; beyond that a workgroup runs too few trials to pay for loading the tables)
constexpr uint32_t kGridPerCu = 128;
// ... and with few simulated GPUs a trial is so short that the tables' load has to be spread over more of them:
// a workgroup runs about three trials at 1 024 GPUs and proportionally more below (12 at 256 GPUs and fewer),
// but the grid never falls below four rounds of resident workgroups (32 per compute unit), so that the last
// round is a small part of the whole.
inline uint32_t trial_grid(uint64_t n_trials, uint32_t n_gpus, int n_cus) {
  const uint64_t most = (uint64_t)n_cus * kGridPerCu, least = (uint64_t)n_cus * 32u;
  const uint64_t scaled = n_trials * n_gpus / (3u * 1024u);
  const uint64_t want = std::min(most, std::max(least, scaled));
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(n_trials, want));
}

thread_local std::string g_error;
int fail(int code, const std::string& msg) {
  g_error = msg;
  return code;
}

// No C++ exception crosses the C boundary.
template <typename F>
int no_throw(F&& body) {
  try {
    return body();
  } catch (...) {
    g_error.clear();  // out of host memory: nothing is allocated to say so
    return LBS_ERR_HIP;
  }
}

struct Params {  // by-value kernel argument
  uint32_t max_len, local_batch, gpus_per_node, n_gpus, snake, stratified;
  uint32_t total;                             // dataset size
  uint32_t guide_words;                       // guide entries the kernel loads (the whole dataset's table, or all strata's)
  uint32_t flagged;                           // some guide entry is flagged: entries have to be looked at for that
  uint32_t turn;                              // 2^32 / n_gpus rounded up: q / n_gpus = umulhi(q, turn) for pool positions q
  uint32_t slot_lo[LBS_MAX_LOCAL_BATCH];      // a GPU's j-th draw: dataset entries before its range (0 / its stratum),
  uint32_t slot_size[LBS_MAX_LOCAL_BATCH];    //   entries in that range,
  uint32_t slot_guide[LBS_MAX_LOCAL_BATCH];   //   where that range's guide table starts in LDS,
  uint32_t slot_base[LBS_MAX_LOCAL_BATCH];    //   and the length below the range's first one
  uint64_t seed, first_trial;
  uint32_t n_trials;
};

// SplitMix64: output number k + 1 of the generator seeded with `seed` is mix(state(seed, k)); the state
// advances by kGamma per draw, so consecutive draws cost one 64-bit addition, not a multiplication.
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t state(uint64_t seed, uint64_t k) { return seed + (k + 1) * kGamma; }
__device__ __forceinline__ uint64_t mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Smallest l in [lo, hi] with counts[l] > index (counts is non-decreasing and counts[hi] > index).
__device__ __forceinline__ uint32_t first_above(const uint32_t* counts, uint32_t lo, uint32_t hi, uint32_t index) {
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (counts[mid] > index) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// Guide entries.  A draw's upper BITS bits select the cell, its other bits are added to the entry, and the sum's upper
// BITS bits are the length (counted from the length below the range's first one): an entry is l * 2^(32 - BITS) for a
// cell that selects l only, and 2^(32 - BITS) - from more for one that selects l + 1 from the lower bits `from` on.
// Entries of kFlagged and above belong to cells that have to be searched: bits 0 .. 9 hold the smallest length minus
// one, bits 10 .. 19 how far the largest one lies above it.  (A mask, an addition and a shift, which issue in two cycles
// each here; comparing with a threshold instead takes three instructions of four cycles.)
template <uint32_t BITS>
constexpr uint32_t kFlagged = ((1u << BITS) - 1u) << (32u - BITS);

// Length selected by the draw with generator state z; `guide` is its range's table, `base` the length below the range's
// first one.  FLAGGED: some entry may be flagged; `range` then says which dataset entries the draw is from.
template <uint32_t BITS, bool FLAGGED, typename F>
__device__ __forceinline__ uint32_t draw(const uint32_t* s_cum, const uint32_t* guide, uint64_t z, uint32_t base, F range) {
  const uint32_t u = (uint32_t)(mix(z) >> 32);
  const uint32_t e = guide[u >> (32u - BITS)];
  uint32_t l = base + ((e + (u & ((1u << (32u - BITS)) - 1u))) >> (32u - BITS));
  if constexpr (FLAGGED) {
    if (e >= kFlagged<BITS>) {
      const uint32_t lo = (e & 1023u) + 1u;
      uint32_t before, size;
      range(before, size);
      l = first_above(s_cum, lo, lo + ((e >> 10) & 1023u), before + __umulhi(u, size));
    }
  }
  return l;
}
// Histogram and guide tables into LDS; returns where the guide tables start.
__device__ __forceinline__ uint32_t* load_tables(uint32_t* s_dyn, const Params& P, const uint32_t* __restrict__ cum,
                                                 const uint32_t* __restrict__ guide) {
  uint32_t* s_guide = s_dyn + P.max_len + 1u;
  for (uint32_t i = threadIdx.x; i <= P.max_len; i += kBlock) s_dyn[i] = cum[i];
  const uint32_t* src = guide + (P.stratified ? kWholeGuideSize : 0u);  // the whole dataset's table comes first
  for (uint32_t i = threadIdx.x; i < P.guide_words; i += kBlock) s_guide[i] = src[i];
  __syncthreads();
  return s_guide;
}

// The value that lane ^ 2^LJ holds.  Within a row of 16 lanes the exchange is a data-parallel move of the
// vector unit (quad permutation, shifts by 4 written to alternate banks of four lanes, rotation by 8);
// across rows it goes through the LDS crossbar.
template <int LJ>
__device__ __forceinline__ uint32_t from_partner(uint32_t x) {
  const int v = (int)x;
  if (LJ == 0) return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
  if (LJ == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);  // quad_perm [2,3,0,1]
  if (LJ == 2) {
    const int t = __builtin_amdgcn_mov_dpp(v, 0x104, 0xf, 0x5, true);            // lanes 0-3, 8-11 of a row read lane + 4
    return (uint32_t)__builtin_amdgcn_update_dpp(t, v, 0x114, 0xf, 0xA, false);  // lanes 4-7, 12-15 read lane - 4
  }
  if (LJ == 3) return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);  // row_ror:8
  return (uint32_t)__shfl_xor(v, 1 << LJ, 64);
}

__device__ __forceinline__ uint32_t partner_of(uint32_t x, int lj) {  // lj is a constant after unrolling
  switch (lj) {
    case 0: return from_partner<0>(x);
    case 1: return from_partner<1>(x);
    case 2: return from_partner<2>(x);
    case 3: return from_partner<3>(x);
    case 4: return from_partner<4>(x);
    default: return from_partner<5>(x);
  }
}

// Sum of x over the lanes that differ from this one only in lane bits lo_bit .. hi_bit - 1 (the same two numbers
// for the whole workgroup): a butterfly, highest bit first, whose steps inside a row of 16 lanes are DPP moves.
// Written as a switch that is entered at the first step and left after the last, so that only the steps
// asked for are executed.
__device__ __forceinline__ uint32_t butterfly_sum(uint32_t x, uint32_t lo_bit, uint32_t hi_bit) {
  if (hi_bit <= lo_bit) return x;
  switch (hi_bit) {
    default: x += from_partner<5>(x); if (lo_bit == 5u) break; [[fallthrough]];
    case 5: x += from_partner<4>(x); if (lo_bit == 4u) break; [[fallthrough]];
    case 4: x += from_partner<3>(x); if (lo_bit == 3u) break; [[fallthrough]];
    case 3: x += from_partner<2>(x); if (lo_bit == 2u) break; [[fallthrough]];
    case 2: x += from_partner<1>(x); if (lo_bit == 1u) break; [[fallthrough]];
    case 1: x += from_partner<0>(x);
  }
  return x;
}

// The value of the lane whose position inside its group of n lanes (n a power of two up to 32) is mirrored.
__device__ __forceinline__ uint32_t from_mirror(uint32_t x, uint32_t n) {
  const int v = (int)x;
  switch (n) {
    case 1: return x;
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
    case 4: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x1B, 0xf, 0xf, true);   // quad_perm [3,2,1,0]
    case 8: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true);  // row_half_mirror
    case 16: return (uint32_t)__builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true); // row_mirror
    default: return (uint32_t)__shfl_xor(v, (int)(n - 1u), 64);
  }
}

// Minimum and maximum over the wavefront, in every lane.
__device__ __forceinline__ void wave_min_max(uint32_t& lo, uint32_t& hi) {
#pragma unroll
  for (int lj = 0; lj < 6; ++lj) {
    lo = min(lo, partner_of(lo, lj));
    hi = max(hi, partner_of(hi, lj));
  }
}

// A workgroup loads the tables once and then runs trials blockIdx.x, blockIdx.x + gridDim.x, ... of the
// call, so the grid need only fill the chip, and thread 0 carries the workgroup's share of the two sums.

// Wavefront minima and maxima of a trial, double-buffered by the parity of the workgroup's trial count: a
// wavefront can be one trial ahead of thread 0, never two (the barrier in between needs all of them).
struct Finish {
  uint32_t lo[2][kWaves], hi[2][kWaves];
};

// Combines the threads' minimum and maximum of trial t (the round-th this workgroup runs); thread 0 stores
// them and adds them to its running sums.
__device__ __forceinline__ void finish_trial(uint32_t lo, uint32_t hi, Finish& f, uint32_t round, uint32_t t,
                                             uint32_t* trial_min, uint32_t* trial_max, unsigned long long& sum_lo,
                                             unsigned long long& sum_hi) {
  wave_min_max(lo, hi);
  const uint32_t buf = round & 1u;
  if ((threadIdx.x & 63u) == 0) f.lo[buf][threadIdx.x >> 6] = lo, f.hi[buf][threadIdx.x >> 6] = hi;
  __syncthreads();
  if (threadIdx.x == 0) {
    lo = min(min(f.lo[buf][0], f.lo[buf][1]), min(f.lo[buf][2], f.lo[buf][3]));
    hi = max(max(f.hi[buf][0], f.hi[buf][1]), max(f.hi[buf][2], f.hi[buf][3]));
    if (trial_min) trial_min[t] = lo;
    if (trial_max) trial_max[t] = hi;
    sum_lo += lo, sum_hi += hi;
  }
}

// Thread 0 adds the workgroup's sums to the call's.
__device__ __forceinline__ void publish_sums(unsigned long long* sums, unsigned long long sum_lo,
                                             unsigned long long sum_hi) {
  if (threadIdx.x == 0) {
    atomicAdd(&sums[0], sum_lo);
    atomicAdd(&sums[1], sum_hi);
  }
}

__global__ __launch_bounds__(64) void k_lbs_clear(unsigned long long* sums) {
  if (threadIdx.x < 2) sums[threadIdx.x] = 0ull;
}

// NONE and STRATIFIED: no redistribution.
template <uint32_t BITS>
__global__ __launch_bounds__(kBlock) void k_lbs_keep(const Params P, const uint32_t* __restrict__ cum,
                                                      const uint32_t* __restrict__ guide, uint32_t* trial_min,
                                                      uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, guide tables
  __shared__ Finish s_finish;
  const uint32_t* s_guide = load_tables(s_dyn, P, cum, guide);
  unsigned long long sum_lo = 0, sum_hi = 0;
  for (uint32_t t = blockIdx.x, round = 0; t < P.n_trials; t += gridDim.x, ++round) {
    const uint64_t k_trial = (P.first_trial + t) * P.n_gpus * (uint64_t)P.local_batch;  // the trial's first draw
    uint32_t lo = 0xffffffffu, hi = 0u;
    const auto draws = [&](auto fl) {
      for (uint32_t g = threadIdx.x; g < P.n_gpus; g += kBlock) {
        uint64_t z = state(P.seed, k_trial + (uint64_t)g * P.local_batch);
        uint32_t tokens = 0;
#pragma unroll 4
        for (uint32_t j = 0; j < P.local_batch; ++j, z += kGamma)
          tokens += draw<BITS, decltype(fl)::value>(
              s_dyn, s_guide + P.slot_guide[j], z, P.slot_base[j],
              [&](uint32_t& before, uint32_t& size) { before = P.slot_lo[j], size = P.slot_size[j]; });
        lo = min(lo, tokens), hi = max(hi, tokens);
      }
    };
    if (P.flagged != 0u) draws(std::true_type{});
    else draws(std::false_type{});
    finish_trial(lo, hi, s_finish, round, t, trial_min, trial_max, sum_lo, sum_hi);
  }
  publish_sums(sums, sum_lo, sum_hi);
}

// Median of three: with c = 0 it is min(a, b), with c = 0xffffffff it is max(a, b) (one v_med3_u32).
__device__ __forceinline__ uint32_t median3(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}

// Sorts the 64 * E values held by a wavefront (value i in v[i / 64] of lane i % 64) into ascending order of i.
// bit[b] is all ones in lanes whose bit b is set and 0 elsewhere (b < 6).
template <int E>
__device__ __forceinline__ void bitonic_sort(uint32_t (&v)[E], const uint32_t (&bit)[6]) {
  constexpr int kLog = 6 + (E == 1 ? 0 : E == 2 ? 1 : E == 4 ? 2 : E == 8 ? 3 : 4);
#pragma unroll
  for (int lk = 1; lk <= kLog; ++lk) {       // merge sorted runs of 2^(lk-1) into runs of k = 2^lk, directions alternating
#pragma unroll
    for (int lj = lk - 1; lj >= 0; --lj) {   // compare-exchange at distance j = 2^lj
      if (lj >= 6) {                         // both entries in this lane
        const int je = 1 << (lj - 6);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if (e & je) continue;
          const bool ascending = ((e >> (lk - 6)) & 1) == 0;  // lk >= 7: the run's direction depends on e alone
          const uint32_t a = v[e], b = v[e | je];
          v[e] = ascending ? min(a, b) : max(a, b);
          v[e | je] = ascending ? max(a, b) : min(a, b);
        }
      } else {                               // the other entry is in lane ^ j
        // The lane with the pair's smaller index keeps the minimum in an ascending run and the maximum in a
        // descending one; the other lane the opposite: `keep` is 0 where the minimum stays, all ones elsewhere.
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const uint32_t descending = lk < 6 ? bit[lk < 6 ? lk : 0] : (((e >> (lk - 6)) & 1) ? 0xffffffffu : 0u);
          const uint32_t keep = bit[lj] ^ descending;
          v[e] = median3(v[e], partner_of(v[e], lj), keep);
        }
      }
    }
  }
}

// LOCAL_RASTER and LOCAL_SNAKE: pool, sort and deal within every node.  E = registers per lane: 64 * E >= the pool.
// IN_LANES: gpus_per_node is a power of two up to 32.  Then sorted entry i = e * 64 + lane lies in column
// lane % gpus_per_node of row e * (64 / gpus_per_node) + lane / gpus_per_node, whose parity is that of
// lane / gpus_per_node for every e, and the deal is a sum within the lane, a mirror exchange inside odd rows
// (snake) and a butterfly over the lane bits above the column: no LDS and no barrier.  Otherwise the sorted
// pool goes to LDS and one lane per GPU walks its column.
template <int E, bool IN_LANES>
__global__ __launch_bounds__(kBlock) void k_lbs_local(const Params P, const uint32_t* __restrict__ cum,
                                                       const uint32_t* __restrict__ guide, uint32_t* trial_min,
                                                       uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, guide tables, (not IN_LANES) one sorted pool per wavefront
  __shared__ Finish s_finish;
  const uint32_t* s_guide = load_tables(s_dyn, P, cum, guide);
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t n_nodes = P.n_gpus / P.gpus_per_node;
  const uint32_t pool = P.gpus_per_node * P.local_batch;
  uint32_t* sorted = s_dyn + P.max_len + 1u + P.guide_words + wave * pool;
  // pool entry i = e * 64 + lane is draw i % local_batch of GPU i / local_batch of the node, for every node alike
  uint32_t base_len[E], goff[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t i = (uint32_t)e * 64u + lane, j = i % P.local_batch;
    const bool real = i < pool;
    base_len[e] = real ? P.slot_base[j] : 0u, goff[e] = real ? P.slot_guide[j] : 0u;
  }
  uint32_t bit[6];
#pragma unroll
  for (int b = 0; b < 6; ++b) bit[b] = 0u - ((lane >> b) & 1u);
  const bool odd_row = ((lane / P.gpus_per_node) & 1u) != 0u;  // IN_LANES only
  const uint32_t gpn_bit = (uint32_t)__ffs((int)P.gpus_per_node) - 1u;  // IN_LANES: gpus_per_node = 2^gpn_bit
  unsigned long long sum_lo = 0, sum_hi = 0;
  for (uint32_t t = blockIdx.x, round = 0; t < P.n_trials; t += gridDim.x, ++round) {
    const uint64_t k_trial = (P.first_trial + t) * P.n_gpus * (uint64_t)P.local_batch;
    uint32_t lo = 0xffffffffu, hi = 0u;
    // Every wavefront makes the same number of rounds, so the barriers below (not IN_LANES) are met by all; a
    // wavefront without a node in the last round only keeps them company.
    for (uint32_t base = 0; base < n_nodes; base += kWaves) {
      const uint32_t node = base + wave;
      const bool active = node < n_nodes;
      if (active) {
        const uint64_t z_node = state(P.seed, k_trial + (uint64_t)node * pool);  // a node's draws are consecutive
        uint32_t v[E];
        const auto draws = [&](auto fl) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const uint32_t i = (uint32_t)e * 64u + lane;
            v[e] = i < pool ? draw<kGuideBits, decltype(fl)::value>(
                                  s_dyn, s_guide + goff[e], z_node + i * kGamma, base_len[e],
                                  [&](uint32_t& before, uint32_t& size) {
                                    before = P.slot_lo[i % P.local_batch], size = P.slot_size[i % P.local_batch];
                                  })
                            : 0xffffffffu;
          }
        };
        if (P.flagged != 0u) draws(std::true_type{});
        else draws(std::false_type{});
        bitonic_sort<E>(v, bit);
        if (IN_LANES) {
          uint32_t tokens = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) tokens += (uint32_t)e * 64u + lane < pool ? v[e] : 0u;  // the padding sorts to the end
          if (P.snake) {  // an odd row is dealt right to left: its column c goes to GPU gpus_per_node - 1 - c
            const uint32_t mirrored = from_mirror(tokens, P.gpus_per_node);
            tokens = odd_row ? mirrored : tokens;
          }
          tokens = butterfly_sum(tokens, gpn_bit, 6u);
          lo = min(lo, tokens), hi = max(hi, tokens);  // every lane now holds the total of GPU lane % gpus_per_node
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const uint32_t i = (uint32_t)e * 64u + lane;
            if (i < pool) sorted[i] = v[e];
          }
        }
      }
      if (!IN_LANES) {
        __syncthreads();
        if (active)
          for (uint32_t c = lane; c < P.gpus_per_node; c += 64u) {
            uint32_t tokens = 0;
            for (uint32_t r = 0; r < P.local_batch; ++r) {
              const uint32_t col = (P.snake && (r & 1u)) ? P.gpus_per_node - 1u - c : c;  // position in the row dealt to GPU c
              tokens += sorted[r * P.gpus_per_node + col];
            }
            lo = min(lo, tokens), hi = max(hi, tokens);
          }
        __syncthreads();
      }
    }
    finish_trial(lo, hi, s_finish, round, t, trial_min, trial_max, sum_lo, sum_hi);
  }
  publish_sums(sums, sum_lo, sum_hi);
}

// Inclusive running sum over the workgroup of one value per thread; all threads call it.  Within a wavefront
// by data-parallel moves, across the four wavefronts through s_scan (kWaves words): one barrier.  The caller leaves s_scan
// alone until the workgroup has passed another barrier (each use in a trial has words of its own).
__device__ __forceinline__ uint32_t block_running_sum(uint32_t* s_scan, uint32_t value) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  uint32_t x = value;
  // within rows of 16 lanes by shifts, then row 0's total to row 1 and row 2's to row 3, then the lower half's to the upper
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
  if (lane == 63u) s_scan[wave] = x;
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < wave; ++w) before += s_scan[w];
  return x + before;
}

// Whole turns round all GPUs in q pool positions: q / n_gpus, as the upper word of a product.  q is at most
// n_gpus * local_batch, so q * n_gpus stays below 2^32 for n_gpus <= kMaxSpreadGpus (or q is a multiple of n_gpus) and
// the quotient is exact.
__device__ __forceinline__ uint32_t turns_of(uint32_t q, const Params& P) {
  return P.n_gpus > 1u ? __umulhi(q, P.turn) : q;
}

// GLOBAL: pool, sort and deal over all GPUs.  The pool is sorted by counting (lengths are small integers):
// after the running sum, the entries of length l hold sorted positions cnt[l-1] .. cnt[l] - 1, and position q
// goes to GPU q % n_gpus.
// SPREAD (n_gpus <= kMaxSpreadGpus): every length adds itself to the GPUs its positions fall on, as a
// difference array over the GPUs: whole turns round all GPUs go to a common base, the rest is a circular
// range [first, first + rest) marked at its two ends; a running sum over the GPUs then gives every GPU's tokens.
// Otherwise every GPU looks up the length at each of its local_batch positions by binary search.
template <bool SPREAD>
__global__ __launch_bounds__(kBlock) void k_lbs_global(const Params P, const uint32_t* __restrict__ cum,
                                                        const uint32_t* __restrict__ guide, uint32_t* trial_min,
                                                        uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, guide table, the trial's own histogram, (SPREAD) one word per GPU
  __shared__ uint32_t s_scan[2][kWaves];
  __shared__ uint32_t s_base;
  __shared__ Finish s_finish;
  const uint32_t* s_guide = load_tables(s_dyn, P, cum, guide);
  uint32_t* s_cnt = s_dyn + P.max_len + 1u + P.guide_words;  // first counts of the trial's draws, then their running sum
  uint32_t* s_gpu = s_cnt + P.max_len + 1u;                           // SPREAD: difference array over the GPUs
  const uint32_t tid = threadIdx.x;
  const uint32_t pool = P.n_gpus * P.local_batch;
  const uint32_t per = (P.max_len + 1u + kBlock - 1u) / kBlock;  // lengths per thread in the running sum
  const uint32_t a = tid * per, b = min(a + per, P.max_len + 1u);
  const uint32_t per_gpu = (P.n_gpus + kBlock - 1u) / kBlock;    // SPREAD: GPUs per thread in theirs
  const uint32_t ga = min(tid * per_gpu, P.n_gpus), gb = min(ga + per_gpu, P.n_gpus);
  unsigned long long sum_lo = 0, sum_hi = 0;
  for (uint32_t t = blockIdx.x, round = 0; t < P.n_trials; t += gridDim.x, ++round) {
    // the previous trial's last reads of s_cnt and s_gpu lie before the barrier in its finish_trial
    for (uint32_t i = tid; i <= P.max_len; i += kBlock) s_cnt[i] = 0u;
    if (SPREAD) {
      for (uint32_t i = tid; i < P.n_gpus; i += kBlock) s_gpu[i] = 0u;
      if (tid == 0) s_base = 0u;
    }
    __syncthreads();
    uint64_t z = state(P.seed, (P.first_trial + t) * (uint64_t)pool + tid);
    const auto draws = [&](auto fl) {
#pragma unroll 4
      for (uint32_t i = tid; i < pool; i += kBlock, z += kBlock * kGamma)
        atomicAdd(&s_cnt[draw<kWholeGuideBits, decltype(fl)::value>(
                      s_dyn, s_guide, z, 0u, [&](uint32_t& before, uint32_t& size) { before = 0u, size = P.total; })],
                  1u);
    };
    if (P.flagged != 0u) draws(std::true_type{});
    else draws(std::false_type{});
    __syncthreads();
    // running sum over lengths: a thread owns a contiguous piece, the pieces' sums are combined across threads
    uint32_t piece = 0;
    for (uint32_t i = a; i < b; ++i) piece += s_cnt[i];
    uint32_t run = block_running_sum(s_scan[0], piece) - piece;  // draws with a length below this thread's piece
    uint32_t lo = 0xffffffffu, hi = 0u;
    if (SPREAD) {
      uint32_t whole_turns = 0;
      for (uint32_t l = a; l < b; ++l) {  // entries of length l: positions run .. run + n - 1
        const uint32_t n = s_cnt[l];
        if (n != 0u) {
          const uint32_t turns = turns_of(n, P), rest = n - turns * P.n_gpus, first = run - turns_of(run, P) * P.n_gpus;
          whole_turns += turns * l;
          if (rest != 0u) {  // unsigned wrap-around is harmless: the sums that are read come out below 2^32
            const uint32_t end = first + rest;
            atomicAdd(&s_gpu[first], l);
            if (end < P.n_gpus) atomicAdd(&s_gpu[end], 0u - l);
            if (end > P.n_gpus) atomicAdd(&s_gpu[0], l), atomicAdd(&s_gpu[end - P.n_gpus], 0u - l);
          }
        }
        run += n;
      }
      if (whole_turns != 0u) atomicAdd(&s_base, whole_turns);
      __syncthreads();
      uint32_t mine = 0;
      for (uint32_t g = ga; g < gb; ++g) mine += s_gpu[g];
      uint32_t tokens = block_running_sum(s_scan[1], mine) - mine + s_base;  // ... of the GPU before this thread's first
      for (uint32_t g = ga; g < gb; ++g) {
        tokens += s_gpu[g];
        lo = min(lo, tokens), hi = max(hi, tokens);
      }
    } else {
      for (uint32_t i = a; i < b; ++i) {
        run += s_cnt[i];
        s_cnt[i] = run;  // draws of length <= i
      }
      __syncthreads();
      for (uint32_t c = tid; c < P.n_gpus; c += kBlock) {
        uint32_t tokens = 0, l = 1;
        for (uint32_t r = 0; r < P.local_batch; ++r) {  // sorted positions r * n_gpus + c grow with r, and so do their lengths
          l = first_above(s_cnt, l, P.max_len, r * P.n_gpus + c);
          tokens += l;
        }
        lo = min(lo, tokens), hi = max(hi, tokens);
      }
    }
    finish_trial(lo, hi, s_finish, round, t, trial_min, trial_max, sum_lo, sum_hi);
  }
  publish_sums(sums, sum_lo, sum_hi);
}

// ---- all five methods on one set of draws ----------------------------------------
// NONE and GLOBAL use the same draws from the whole dataset, STRATIFIED and the two LOCAL methods the same
// stratified draws (draw number k of a run does not depend on the method), so one pass makes each set once:
// first a thread per GPU draws from the whole dataset, sums its GPU's tokens (NONE) and counts the lengths
// for the counting sort (GLOBAL, as in k_lbs_global<true>); then a wavefront per node draws the stratified
// pool into registers, adds up each GPU's own draws (STRATIFIED: local_batch consecutive pool entries, a
// butterfly over the low lane bits), sorts and deals twice (LOCAL_RASTER, LOCAL_SNAKE, as in
// k_lbs_local<E, true>).  Needs gpus_per_node and local_batch to be powers of two (<= 32 and <= 64).
constexpr uint32_t kMethods = 5;

// One trial's draws from the whole dataset: NONE (a thread per GPU sums its draws) and GLOBAL (the lengths are counted,
// then as in k_lbs_global<true>).  All threads of the workgroup call it; s_cnt, s_gpu, *s_base and s_scan are its own until
// the next barrier of the caller.
__device__ __forceinline__ void whole_draws(const Params& P, const uint32_t* s_cum, const uint32_t* s_whole, uint32_t* s_cnt,
                                            uint32_t* s_gpu, uint32_t* s_base, uint32_t (*s_scan)[kWaves], uint64_t k_trial,
                                            uint32_t& none_lo, uint32_t& none_hi, uint32_t& glob_lo, uint32_t& glob_hi) {
  const uint32_t tid = threadIdx.x;
  const uint32_t per = (P.max_len + 1u + kBlock - 1u) / kBlock;
  const uint32_t a = tid * per, b = min(a + per, P.max_len + 1u);
  const uint32_t per_gpu = (P.n_gpus + kBlock - 1u) / kBlock;
  const uint32_t ga = min(tid * per_gpu, P.n_gpus), gb = min(ga + per_gpu, P.n_gpus);
  for (uint32_t i = tid; i <= P.max_len; i += kBlock) s_cnt[i] = 0u;
  for (uint32_t i = tid; i < P.n_gpus; i += kBlock) s_gpu[i] = 0u;
  if (tid == 0) *s_base = 0u;
  __syncthreads();
  const auto draws = [&](auto fl) {
    for (uint32_t g = tid; g < P.n_gpus; g += kBlock) {
      uint64_t z = state(P.seed, k_trial + (uint64_t)g * P.local_batch);
      uint32_t tokens = 0;
#pragma unroll 4
      for (uint32_t j = 0; j < P.local_batch; ++j, z += kGamma) {
        const uint32_t l = draw<kWholeGuideBits, decltype(fl)::value>(
            s_cum, s_whole, z, 0u, [&](uint32_t& before, uint32_t& size) { before = 0u, size = P.total; });
        tokens += l;
        atomicAdd(&s_cnt[l], 1u);
      }
      none_lo = min(none_lo, tokens), none_hi = max(none_hi, tokens);
    }
  };
  if (P.flagged != 0u) draws(std::true_type{});
  else draws(std::false_type{});
  __syncthreads();
  {
    uint32_t piece = 0;
    for (uint32_t i = a; i < b; ++i) piece += s_cnt[i];
    uint32_t run = block_running_sum(s_scan[0], piece) - piece;
    uint32_t whole_turns = 0;
    for (uint32_t l = a; l < b; ++l) {
      const uint32_t n = s_cnt[l];
      if (n != 0u) {
        const uint32_t turns = turns_of(n, P), rest = n - turns * P.n_gpus, first = run - turns_of(run, P) * P.n_gpus;
        whole_turns += turns * l;
        if (rest != 0u) {
          const uint32_t end = first + rest;
          atomicAdd(&s_gpu[first], l);
          if (end < P.n_gpus) atomicAdd(&s_gpu[end], 0u - l);
          if (end > P.n_gpus) atomicAdd(&s_gpu[0], l), atomicAdd(&s_gpu[end - P.n_gpus], 0u - l);
        }
      }
      run += n;
    }
    if (whole_turns != 0u) atomicAdd(s_base, whole_turns);
    __syncthreads();
    uint32_t mine = 0;
    for (uint32_t g = ga; g < gb; ++g) mine += s_gpu[g];
    uint32_t tokens = block_running_sum(s_scan[1], mine) - mine + *s_base;
    for (uint32_t g = ga; g < gb; ++g) {
      tokens += s_gpu[g];
      glob_lo = min(glob_lo, tokens), glob_hi = max(glob_hi, tokens);
    }
  }
}

struct FinishAll {
  uint32_t lo[2][kMethods][kWaves], hi[2][kMethods][kWaves];
};

template <int E>
__global__ __launch_bounds__(kBlock, E <= 2 ? 6 : E == 4 ? 4 : E == 8 ? 3 : 2) void k_lbs_all(const Params P, const uint32_t* __restrict__ cum,
                                                     const uint32_t* __restrict__ guide, uint32_t* trial_min,
                                                     uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, all guide tables, the trial's own histogram, one word per GPU
  __shared__ uint32_t s_scan[2][kWaves];
  __shared__ uint32_t s_base;
  __shared__ FinishAll s_fin;
  __shared__ unsigned long long s_sum[2u * kMethods];  // the workgroup's share of the sums: thread i keeps sum i
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  if (tid < 2u * kMethods) s_sum[tid] = 0ull;
  uint32_t* s_whole = s_dyn + P.max_len + 1u;          // guide table of the whole dataset
  uint32_t* s_strata = s_whole + kWholeGuideSize;      // guide tables of the strata
  uint32_t* s_cnt = s_whole + P.guide_words;
  uint32_t* s_gpu = s_cnt + P.max_len + 1u;
  for (uint32_t i = tid; i <= P.max_len; i += kBlock) s_dyn[i] = cum[i];
  for (uint32_t i = tid; i < P.guide_words; i += kBlock) s_whole[i] = guide[i];
  __syncthreads();

  const uint32_t pool_all = P.n_gpus * P.local_batch;
  const uint32_t n_nodes = P.n_gpus / P.gpus_per_node;
  const uint32_t pool = P.gpus_per_node * P.local_batch;
  uint32_t base_len[E], goff[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t i = (uint32_t)e * 64u + lane, j = i % P.local_batch;
    const bool real = i < pool;
    base_len[e] = real ? P.slot_base[j] : 0u, goff[e] = real ? P.slot_guide[j] : 0u;
  }
  uint32_t bit[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) bit[q] = 0u - ((lane >> q) & 1u);
  const bool odd_row = ((lane / P.gpus_per_node) & 1u) != 0u;
  const uint32_t gpn_bit = (uint32_t)__ffs((int)P.gpus_per_node) - 1u, batch_bit = (uint32_t)__ffs((int)P.local_batch) - 1u;

  for (uint32_t t = blockIdx.x, round = 0; t < P.n_trials; t += gridDim.x, ++round) {
    const uint32_t buf = round & 1u;
    uint32_t lo[kMethods], hi[kMethods];
#pragma unroll
    for (uint32_t q = 0; q < kMethods; ++q) lo[q] = 0xffffffffu, hi[q] = 0u;
    const uint64_t k_trial = (P.first_trial + t) * (uint64_t)pool_all;  // the trial's first draw
    whole_draws(P, s_dyn, s_whole, s_cnt, s_gpu, &s_base, s_scan, k_trial, lo[LBS_NONE], hi[LBS_NONE], lo[LBS_GLOBAL],
                hi[LBS_GLOBAL]);
    // these two are filed now, so that they need no registers during the sort
    wave_min_max(lo[LBS_NONE], hi[LBS_NONE]);
    wave_min_max(lo[LBS_GLOBAL], hi[LBS_GLOBAL]);
    if (lane == 0) {
      s_fin.lo[buf][LBS_NONE][wave] = lo[LBS_NONE], s_fin.hi[buf][LBS_NONE][wave] = hi[LBS_NONE];
      s_fin.lo[buf][LBS_GLOBAL][wave] = lo[LBS_GLOBAL], s_fin.hi[buf][LBS_GLOBAL][wave] = hi[LBS_GLOBAL];
    }
    // ---- stratified draws, a wavefront per node: STRATIFIED, LOCAL_RASTER, LOCAL_SNAKE (no LDS writes, no barriers)
    for (uint32_t node = wave; node < n_nodes; node += kWaves) {
      const uint64_t z_node = state(P.seed, k_trial + (uint64_t)node * pool);
      uint32_t v[E];
      const auto draws = [&](auto fl) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const uint32_t i = (uint32_t)e * 64u + lane;
          v[e] = i < pool ? draw<kGuideBits, decltype(fl)::value>(
                                s_dyn, s_strata + goff[e], z_node + i * kGamma, base_len[e],
                                [&](uint32_t& before, uint32_t& size) {
                                  before = P.slot_lo[i % P.local_batch], size = P.slot_size[i % P.local_batch];
                                })
                          : 0xffffffffu;
        }
      };
      if (P.flagged != 0u) draws(std::true_type{});
      else draws(std::false_type{});
#pragma unroll
      for (int e = 0; e < E; ++e) {  // a GPU's own draws are local_batch consecutive pool entries
        const bool real = (uint32_t)e * 64u + lane < pool;
        const uint32_t own = butterfly_sum(real ? v[e] : 0u, 0u, batch_bit);
        if (real) lo[LBS_STRATIFIED] = min(lo[LBS_STRATIFIED], own), hi[LBS_STRATIFIED] = max(hi[LBS_STRATIFIED], own);
      }
      bitonic_sort<E>(v, bit);
      uint32_t column = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) column += (uint32_t)e * 64u + lane < pool ? v[e] : 0u;
      const uint32_t mirrored = from_mirror(column, P.gpus_per_node);
      const uint32_t raster = butterfly_sum(column, gpn_bit, 6u);
      const uint32_t snake = butterfly_sum(odd_row ? mirrored : column, gpn_bit, 6u);
      lo[LBS_LOCAL_RASTER] = min(lo[LBS_LOCAL_RASTER], raster), hi[LBS_LOCAL_RASTER] = max(hi[LBS_LOCAL_RASTER], raster);
      lo[LBS_LOCAL_SNAKE] = min(lo[LBS_LOCAL_SNAKE], snake), hi[LBS_LOCAL_SNAKE] = max(hi[LBS_LOCAL_SNAKE], snake);
    }
    // ---- the trial's five results
#pragma unroll
    for (uint32_t q = LBS_STRATIFIED; q <= LBS_LOCAL_SNAKE; ++q) {
      wave_min_max(lo[q], hi[q]);
      if (lane == 0) s_fin.lo[buf][q][wave] = lo[q], s_fin.hi[buf][q][wave] = hi[q];
    }
    __syncthreads();  // also: this trial's last reads of s_cnt and s_gpu lie before the next trial's clearing
    if (tid < 2u * kMethods) {  // thread 2 q: method q's minimum; thread 2 q + 1: its maximum
      const uint32_t q = tid >> 1;
      uint32_t r;
      if (tid & 1u) {
        r = max(max(s_fin.hi[buf][q][0], s_fin.hi[buf][q][1]), max(s_fin.hi[buf][q][2], s_fin.hi[buf][q][3]));
        if (trial_max) trial_max[(size_t)q * P.n_trials + t] = r;
      } else {
        r = min(min(s_fin.lo[buf][q][0], s_fin.lo[buf][q][1]), min(s_fin.lo[buf][q][2], s_fin.lo[buf][q][3]));
        if (trial_min) trial_min[(size_t)q * P.n_trials + t] = r;
      }
      s_sum[tid] += r;
    }
  }
  if (tid < 2u * kMethods) atomicAdd(&sums[tid], s_sum[tid]);
}

// ---- node-local methods with the strata in bins ------------------------------------
// A stratum's entries of a node's pool are gpus_per_node * quota of its sorted entries, i.e. `quota` whole rows of the
// deal, whatever the draws: sorted row j holds what the GPUs' j-th draws (counted stratum by stratum) sort to.  So the
// strata can be sorted apart, in any place, as long as each row's parity (snake) is that of its j.  The host packs
// them into bins of 64 entries, 64 / gpus_per_node rows each, strata ascending in a bin, so that sorting a bin sorts its
// strata.  Entries are 16-bit halves of a register: BINS == 2, the two bins of a node; BINS == 1, two nodes whose strata
// all fit in one bin.  Row r's entry in column c is drawn by GPU c, so that before the sort the column sums are what
// every GPU drew itself (STRATIFIED).
//   Sorting 64 instead of 128 entries takes 21 stages instead of 28, and a packed stage across lanes takes three
// instructions for two entries where bitonic_sort<2> takes five.  The bound is vector issue: 32-bit logic, shifts and
// additions take two cycles a wavefront, everything else here (minima, moves across lanes, multiplications) four.
//   LG > 0: gpus_per_node = 2^LG; column c of a row lies in register c of one lane, a bin in 2^(6 - LG) lanes, and a
// wavefront sorts 2^LG nodes (BINS == 1: twice as many) at a time: 15 of the 21 stages (nodes of 8) then pair registers of one lane, at
// 2 instead of 5 cycles an entry, and a row is mirrored by naming its registers backwards.  Needs as many nodes as
// that, else lanes would idle.  LG == 0: any power of two up to 16; a bin lies in the 64 lanes, one node at a time.
//   Measured (100 000 trials of 1 024 GPUs x 16, nodes of 8, five methods at once): 3.11 ms; one node at a time (LG == 0)
// with thresholds compared 3.90; k_lbs_all<2>, whose draws were all searched, 5.31.  20 000 trials: snake alone 420 us
// (k_lbs_local 637), nodes of 4: 688 (1168), 8 sequences a GPU: 351 (596), 64 GPUs: 158 (187).
// A run of many short trials (one node a wavefront at most, and its strata fit in one bin) is better off with k_lbs_local, of
// which eight workgroups are resident instead of six, once a workgroup runs this many of them; up to there its longer start
// decides.  One node of 8, batch 8: 20 000 trials 110 us (k_lbs_local 207), 200 000 165 (243), 1 500 000 928 (826); four nodes of
// 2, batch 4: 110 (207), 181 (265), 1 160 (1 106).
constexpr uint32_t kBinsMostShortTrials = 60;
struct Bins {
  uint8_t slot[2][64];  // slot (draw number j of a GPU) whose stratum row r of the bin belongs to, or kNoSlot: padding
  uint32_t count;       // bins used: 1 or 2; 0: the strata do not fit
  uint32_t padded;      // some row is padding
};
constexpr uint8_t kNoSlot = 255;

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t min_halves(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t max_halves(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Sorts the low halves, and the high halves, of every group of 2^(6 - LG) lanes: entry p of a group's 64 is in register
// p % 2^LG of its lane p / 2^LG; ascending order of p (bitonic network, merges of 2^lk entries, distances 2^lj).
//   Distances below 2^LG pair two registers of a lane.  In a stage across lanes one lane of a pair keeps the minimum
// and the other the maximum; a lane that is to keep the maximum holds complements: the maximum is then a minimum too,
// and as its partner's values are complemented exactly when its own are not, both keep min(own, ~partner's).  A lane
// whose run descends holds complements while it pairs its registers, too.  Between stages, lanes change from one form to
// the other where `bit` masks say so (bit[b]: all ones in lanes whose bit b is set).
template <int LG>
__device__ __forceinline__ void sort_halves(uint32_t (&v)[1 << LG], const uint32_t (&bit)[6]) {
  constexpr int R = 1 << LG;
  uint32_t form = 0;  // which lanes hold complements now; all of this folds into a few masks
#pragma unroll
  for (int lk = 1; lk <= 6; ++lk) {
    const uint32_t descends = (lk >= LG && lk < 6) ? bit[lk - LG] : 0u;  // lk < LG: by register, below
#pragma unroll
    for (int lj = lk - 1; lj >= 0; --lj) {
      const uint32_t want = lj >= LG ? descends ^ bit[lj - LG] : descends;
      const uint32_t change = form ^ want;
      // the first register stage of a merge follows a lane stage or another merge; later ones need no change
      const bool changes = lj >= LG || lj == lk - 1 || lj == LG - 1;
      if (changes) {
#pragma unroll
        for (int c = 0; c < R; ++c) v[c] ^= change;
        form = want;
      }
      if (lj >= LG) {
#pragma unroll
        for (int c = 0; c < R; ++c) v[c] = min_halves(v[c], ~partner_of(v[c], lj - LG));
      } else {
#pragma unroll
        for (int c = 0; c < R; ++c) {
          const int d = c ^ (1 << lj);
          if (d < c) continue;
          const bool down = lk < LG && ((c >> lk) & 1) != 0;
          const uint32_t x = min_halves(v[c], v[d]), y = max_halves(v[c], v[d]);
          v[c] = down ? y : x, v[d] = down ? x : y;
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < R; ++c) v[c] ^= form;
}

// Sums of the R = 2^LG columns over a group's 2^(6 - LG) rows (lanes), halves apart; which lane ends up with which
// column does not matter.  Lanes of a pair share the columns between them while there are several, then each adds up
// its own.  sel[b]: all ones in lanes whose bit b is set.
template <int LG>
__device__ __forceinline__ uint32_t column_sums(uint32_t (&x)[1 << LG], const uint32_t (&sel)[6]) {
  static_assert(LG <= 3, "a group needs as many lanes as columns");
#pragma unroll
  for (int b = 0; b < 6 - LG; ++b) {
    const int n = (1 << LG) >> (b + 1);  // columns a lane is left with after this step
    if (n == 0) {
      x[0] += partner_of(x[0], b);
      continue;
    }
#pragma unroll
    for (int c = 0; c < n; ++c) {
      const uint32_t keep = (x[c] & ~sel[b]) | (x[c + n] & sel[b]);
      const uint32_t send = (x[c + n] & ~sel[b]) | (x[c] & sel[b]);
      x[c] = keep + partner_of(send, b);
    }
  }
  return x[0];
}

template <int LG, int BINS, bool WHOLE>
__global__ __launch_bounds__(kBlock, 6) void k_lbs_bins(const Params P, const Bins L, const uint32_t method,
                                                         const uint32_t* __restrict__ cum, const uint32_t* __restrict__ guide,
                                                         uint32_t* trial_min, uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, guide tables; WHOLE: the trial's own histogram, one word per GPU
  __shared__ uint32_t s_scan[2][kWaves];
  __shared__ uint32_t s_base;
  __shared__ FinishAll s_fin;
  __shared__ unsigned long long s_sum[2u * kMethods];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < 2u * kMethods) s_sum[tid] = 0ull;
  uint32_t* s_whole = s_dyn + P.max_len + 1u;
  uint32_t* s_strata = s_whole + (WHOLE ? kWholeGuideSize : 0u);
  uint32_t* s_cnt = s_whole + P.guide_words;
  uint32_t* s_gpu = s_cnt + P.max_len + 1u;
  for (uint32_t i = tid; i <= P.max_len; i += kBlock) s_dyn[i] = cum[i];
  for (uint32_t i = tid; i < P.guide_words; i += kBlock) s_whole[i] = guide[i + (WHOLE ? 0u : kWholeGuideSize)];
  __syncthreads();

  constexpr int R = 1 << LG;  // columns a lane holds
  const uint32_t pool_all = P.n_gpus * P.local_batch;
  const uint32_t n_nodes = P.n_gpus / P.gpus_per_node;
  const uint32_t pool = P.gpus_per_node * P.local_batch;
  const uint32_t gpn_bit = LG > 0 ? (uint32_t)LG : (uint32_t)__ffs((int)P.gpus_per_node) - 1u;  // gpus_per_node = 2^gpn_bit
  const uint32_t row = LG > 0 ? lane & ((1u << (6 - LG)) - 1u) : lane >> gpn_bit;
  const uint32_t column = LG > 0 ? 0u : lane & (P.gpus_per_node - 1u);  // of the lane's first register
  const uint32_t group = LG > 0 ? lane >> (6 - LG) : 0u;                // which of the wavefront's nodes
  uint32_t bit[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) bit[q] = 0u - ((lane >> q) & 1u);
  uint32_t real = 0, odd = 0, slot[2], base_len[2], goff[2];
  uint64_t step[2];
  constexpr uint32_t kNodes = R * (BINS == 2 ? 1u : 2u);  // nodes a wavefront takes at a time
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t j = L.slot[BINS == 2 ? h : 0][row];
    const uint32_t half = h == 0 ? 0xffffu : 0xffff0000u;
    if (j != kNoSlot) real |= half;
    if (j != kNoSlot && (j & 1u)) odd |= half;
    slot[h] = j != kNoSlot ? j : 0u;
    base_len[h] = P.slot_base[slot[h]], goff[h] = P.slot_guide[slot[h]];
    const uint32_t node = BINS == 2 ? group : group * 2u + (uint32_t)h;
    step[h] = (uint64_t)(node * pool + column * P.local_batch + slot[h]) * kGamma;
  }
  const uint64_t next_column = (uint64_t)P.local_batch * kGamma;

  for (uint32_t t = blockIdx.x, round = 0; t < P.n_trials; t += gridDim.x, ++round) {
    const uint32_t buf = round & 1u;
    const uint64_t k_trial = (P.first_trial + t) * (uint64_t)pool_all;
    if (WHOLE) {
      uint32_t none_lo = 0xffffffffu, none_hi = 0u, glob_lo = 0xffffffffu, glob_hi = 0u;
      whole_draws(P, s_dyn, s_whole, s_cnt, s_gpu, &s_base, s_scan, k_trial, none_lo, none_hi, glob_lo, glob_hi);
      wave_min_max(none_lo, none_hi);
      wave_min_max(glob_lo, glob_hi);
      if (lane == 0) {
        s_fin.lo[buf][LBS_NONE][wave] = none_lo, s_fin.hi[buf][LBS_NONE][wave] = none_hi;
        s_fin.lo[buf][LBS_GLOBAL][wave] = glob_lo, s_fin.hi[buf][LBS_GLOBAL][wave] = glob_hi;
      }
    }
    // Running minima and maxima: LG > 0, of own, raster, snake in turn; LG == 0, one for all three, told apart by the lane.
    // BINS == 1: 16-bit halves.
    constexpr int M = LG > 0 ? 3 : 1;
    uint32_t lo[M], hi[M];
#pragma unroll
    for (int m = 0; m < M; ++m) lo[m] = 0xffffffffu, hi[m] = 0u;
    for (uint32_t first = wave * kNodes; first < n_nodes; first += kWaves * kNodes) {
      const uint64_t z0 = state(P.seed, k_trial + (uint64_t)first * pool);
      uint32_t v[R];
      const auto draws = [&](auto fl) {
#pragma unroll
        for (int c = 0; c < R; ++c) {
          uint32_t d[2];
#pragma unroll
          for (int h = 0; h < 2; ++h)
            d[h] = draw<kGuideBits, decltype(fl)::value>(
                s_dyn, s_strata + goff[h], z0 + (uint64_t)c * next_column + step[h], base_len[h],
                [&](uint32_t& before, uint32_t& size) { before = P.slot_lo[slot[h]], size = P.slot_size[slot[h]]; });
          v[c] = d[0] | (d[1] << 16);
        }
      };
      if (P.flagged != 0u) draws(std::true_type{});
      else draws(std::false_type{});
      if (first + kNodes > n_nodes) {  // the last nodes: others take the place of those that are not there
        const uint32_t node = first + (BINS == 2 ? group : group * 2u);
        // BINS == 1: a second node that is not there repeats the first; a whole group that is not there is left out below
        if (BINS == 1 && node + 1u >= n_nodes) {
#pragma unroll
          for (int c = 0; c < R; ++c) v[c] = (v[c] & 0xffffu) | (v[c] << 16);
        }
      }
      const bool there = LG == 0 || first + (BINS == 2 ? group : group * 2u) < n_nodes;
      uint32_t own[R];
#pragma unroll
      for (int c = 0; c < R; ++c) own[c] = v[c];
      if (L.padded != 0u) {
        // 0xffff sorts behind every length, into the bin's last rows: again the padded ones
#pragma unroll
        for (int c = 0; c < R; ++c) own[c] &= real, v[c] |= ~real;
      }
      uint32_t sum[3];
      if constexpr (LG > 0) sum[0] = column_sums<LG>(own, bit);
      else sum[0] = own[0];
      sort_halves<LG>(v, bit);
      if (L.padded != 0u) {
#pragma unroll
        for (int c = 0; c < R; ++c) v[c] &= real;
      }
      if constexpr (LG > 0) {
        uint32_t snake[R];
#pragma unroll
        for (int c = 0; c < R; ++c) snake[c] = (v[c] & ~odd) | (v[R - 1 - c] & odd);
        sum[1] = column_sums<LG>(v, bit);
        sum[2] = column_sums<LG>(snake, bit);
      } else {
        sum[1] = v[0];
        const uint32_t mirrored = from_mirror(v[0], P.gpus_per_node);
        sum[2] = (v[0] & ~odd) | (mirrored & odd);
      }
      if (BINS == 2) {
#pragma unroll
        for (int m = 0; m < 3; ++m) sum[m] = (sum[m] & 0xffffu) + (sum[m] >> 16);
      }
      if constexpr (LG > 0) {
        if (there) {
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            lo[m] = BINS == 2 ? min(lo[m], sum[m]) : min_halves(lo[m], sum[m]);
            hi[m] = BINS == 2 ? max(hi[m], sum[m]) : max_halves(hi[m], sum[m]);
          }
        }
      } else {
        // sums over the rows of 16 lanes: row 0 ends up with `own`, row 2 with `raster`, rows 1 and 3 with `snake`
        const auto p = __builtin_amdgcn_permlane32_swap(sum[0], sum[1], false, false);
        const auto q = __builtin_amdgcn_permlane32_swap(sum[2], sum[2], false, false);
        const auto r = __builtin_amdgcn_permlane16_swap(p[0] + p[1], q[0] + q[1], false, false);
        const uint32_t tokens = butterfly_sum(r[0] + r[1], gpn_bit, 4u);
        lo[0] = BINS == 2 ? min(lo[0], tokens) : min_halves(lo[0], tokens);
        hi[0] = BINS == 2 ? max(hi[0], tokens) : max_halves(hi[0], tokens);
      }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (BINS == 1) {  // 0xffffffff: a lane that has seen no node
        lo[m] = lo[m] == 0xffffffffu ? lo[m] : min(lo[m] & 0xffffu, lo[m] >> 16);
        hi[m] = max(hi[m] & 0xffffu, hi[m] >> 16);
      }
#pragma unroll
      for (int lj = 0; lj < (LG > 0 ? 6 : 4); ++lj) lo[m] = min(lo[m], partner_of(lo[m], lj)), hi[m] = max(hi[m], partner_of(hi[m], lj));
      if (LG > 0 ? lane == 0u : (lane & 15u) == 0u && lane < 48u) {
        const uint32_t which = LG > 0 ? (uint32_t)m : lane == 0u ? 0u : lane == 16u ? 2u : 1u;
        const uint32_t q = which == 0u ? LBS_STRATIFIED : which == 1u ? LBS_LOCAL_RASTER : LBS_LOCAL_SNAKE;
        s_fin.lo[buf][q][wave] = lo[m], s_fin.hi[buf][q][wave] = hi[m];
      }
    }
    __syncthreads();  // also: this trial's last reads of s_cnt and s_gpu lie before the next trial's clearing
    if (tid < 2u * kMethods) {  // thread 2 q: method q's minimum; thread 2 q + 1: its maximum
      const uint32_t m = tid >> 1;
      if (WHOLE || m == method) {
        const size_t at = WHOLE ? (size_t)m * P.n_trials + t : t;
        uint32_t x;
        if (tid & 1u) {
          x = max(max(s_fin.hi[buf][m][0], s_fin.hi[buf][m][1]), max(s_fin.hi[buf][m][2], s_fin.hi[buf][m][3]));
          if (trial_max) trial_max[at] = x;
        } else {
          x = min(min(s_fin.lo[buf][m][0], s_fin.lo[buf][m][1]), min(s_fin.lo[buf][m][2], s_fin.lo[buf][m][3]));
          if (trial_min) trial_min[at] = x;
        }
        s_sum[tid] += x;
      }
    }
  }
  if (tid < 2u * kMethods && (WHOLE || (tid >> 1) == method)) atomicAdd(&sums[WHOLE ? tid : (tid & 1u)], s_sum[tid]);
}

// k_lbs_bins for a run whose strata fit in L.count bins.  Columns in registers for nodes of 4 and 8: with two columns only 6 of the
// 21 stages would stay within a lane (11 with four, 15 with eight), and sixteen are more columns than a group has lanes.
template <bool WHOLE>
auto pick_bins(const Bins& L, uint32_t gpus_per_node, uint32_t n_nodes) {
  const bool two = L.count == 2;
  if (n_nodes >= gpus_per_node * (two ? 1u : 2u)) {
    if (gpus_per_node == 4) return two ? k_lbs_bins<2, 2, WHOLE> : k_lbs_bins<2, 1, WHOLE>;
    if (gpus_per_node == 8) return two ? k_lbs_bins<3, 2, WHOLE> : k_lbs_bins<3, 1, WHOLE>;
  }
  return two ? k_lbs_bins<0, 2, WHOLE> : k_lbs_bins<0, 1, WHOLE>;
}

__global__ __launch_bounds__(64) void k_lbs_clear_all(unsigned long long* sums) {
  if (threadIdx.x < 2u * kMethods) sums[threadIdx.x] = 0ull;
}

// Guide table of the `size` entries after the first `before` (lengths base + 1 and up).  The index a draw selects
// grows with the draw, and the length with the index, so a cell's two ends bound everything between.  Returns
// whether some entry is flagged.
template <uint32_t BITS>
bool fill_guide(uint32_t* out, const std::vector<uint32_t>& cum, uint32_t before, uint32_t size, uint32_t base) {
  bool flagged = false;
  constexpr uint32_t kLow = 32u - BITS;
  uint32_t l = base + 1u;  // cells and their ends come in ascending order, and so do the lengths
  const auto length_of = [&](uint32_t index) {  // smallest length with more than `index` entries up to it
    while (cum[l] <= index) ++l;
    return l;
  };
  for (uint32_t ub = 0; ub < (1u << BITS); ++ub) {
    const uint64_t u_min = (uint64_t)ub << kLow, u_max = u_min + (1ull << kLow) - 1u;
    if (size == 0) {
      out[ub] = 0u;  // never drawn from
      continue;
    }
    const uint32_t l_min = length_of(before + (uint32_t)((u_min * size) >> 32));
    const uint32_t l_max = length_of(before + (uint32_t)((u_max * size) >> 32));
    if (l_max > l_min + 1u || l_max - base >= (1u << BITS) - 1u) {
      out[ub] = kFlagged<BITS> | (l_min - 1u) | ((l_max - l_min) << 10);
      flagged = true;
      continue;
    }
    out[ub] = (l_min - base) << kLow;
    if (l_max > l_min) {  // the first draw whose index reaches the entries of l_max
      const uint64_t from = (((uint64_t)(cum[l_min] - before) << 32) + size - 1u) / size;
      out[ub] += (uint32_t)((1ull << kLow) - (from - u_min));
    }
  }
  return flagged;
}

// Measurement only: how many lane-operations per second the vector units issue for the instruction kinds the
// simulation is made of.  Pure register arithmetic on eight independent chains per lane (enough to cover every
// instruction's latency), one store per thread at the end so that nothing is optimised away.
template <int KIND>
__global__ __launch_bounds__(256) void k_issue_probe(uint32_t* out, uint32_t iters, uint32_t seed) {
  uint32_t a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = seed * (i + 1) + threadIdx.x;
  const uint32_t c = seed | 1u;
  for (uint32_t it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (KIND == LBS_PROBE_XOR_ADD) a[i] = (a[i] ^ c) + 0x9E3779B9u;
      if (KIND == LBS_PROBE_MUL_LO) a[i] = a[i] * 0x85EBCA6Bu + 1u;
      if (KIND == LBS_PROBE_MUL_HI_ADD) a[i] = __umulhi(a[i], c) + a[i];
      if (KIND == LBS_PROBE_MED3) a[i] = max(min(a[i], c), min(max(a[i], c), it));
      if (KIND == LBS_PROBE_DPP_ADD)
        a[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)a[i], (int)a[i], 0xB1, 0xf, 0xf, false) + 1u;
      if (KIND == LBS_PROBE_BPERMUTE_ADD) a[i] = (uint32_t)__shfl_xor((int)a[i], 16, 64) + 1u;
      if (KIND == LBS_PROBE_FMA_F32) a[i] = __float_as_uint(__fmaf_rn(__uint_as_float(a[i]), 1.0001f, 0.5f));
    }
  }
  uint32_t r = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) r ^= a[i];
  out[(size_t)blockIdx.x * 256 + threadIdx.x] = r;
}

}  // namespace
}  // namespace lbs

using namespace lbs;

extern "C" {

const char* lbs_last_error(void) { return g_error.c_str(); }

int lbs_issue_rate_probe(int kind, uint32_t n_workgroups, uint32_t iters, uint32_t* out, void* stream) {
  if (!out) return fail(LBS_ERR_NULL, "out is NULL");
  if (n_workgroups == 0 || n_workgroups > (1u << 20)) return fail(LBS_ERR_ARG, "n_workgroups must lie in [1, 2^20]");
  void (*kernel)(uint32_t*, uint32_t, uint32_t) = nullptr;
  switch (kind) {
    case LBS_PROBE_XOR_ADD: kernel = k_issue_probe<LBS_PROBE_XOR_ADD>; break;
    case LBS_PROBE_MUL_LO: kernel = k_issue_probe<LBS_PROBE_MUL_LO>; break;
    case LBS_PROBE_MUL_HI_ADD: kernel = k_issue_probe<LBS_PROBE_MUL_HI_ADD>; break;
    case LBS_PROBE_MED3: kernel = k_issue_probe<LBS_PROBE_MED3>; break;
    case LBS_PROBE_DPP_ADD: kernel = k_issue_probe<LBS_PROBE_DPP_ADD>; break;
    case LBS_PROBE_BPERMUTE_ADD: kernel = k_issue_probe<LBS_PROBE_BPERMUTE_ADD>; break;
    case LBS_PROBE_FMA_F32: kernel = k_issue_probe<LBS_PROBE_FMA_F32>; break;
    default: return fail(LBS_ERR_ARG, "unknown probe kind");
  }
  hipLaunchKernelGGL(kernel, dim3(n_workgroups), dim3(256), 0, (hipStream_t)stream, out, iters, 12345u);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LBS_ERR_HIP, std::string("launching the probe: ") + hipGetErrorString(e));
  return 0;
}

static int dataset_create(lbs_dataset** out, int device, uint32_t max_len, const uint32_t* cum, uint32_t n_strata,
                          const uint32_t* stratum_end) {
  if (!out) return fail(LBS_ERR_NULL, "out is NULL");
  *out = nullptr;
  if (!cum || !stratum_end) return fail(LBS_ERR_NULL, "cum or stratum_end is NULL");
  if (max_len == 0 || n_strata == 0) return fail(LBS_ERR_ARG, "max_len and n_strata must be positive");
  if (max_len > LBS_MAX_LEN) return fail(LBS_ERR_LIMIT, "max_len exceeds LBS_MAX_LEN");
  if (n_strata > LBS_MAX_STRATA) return fail(LBS_ERR_LIMIT, "n_strata exceeds LBS_MAX_STRATA");
  if (device < -1) return fail(LBS_ERR_ARG, "device must be >= 0, or -1 for a host-only dataset");
  if (cum[0] != 0) return fail(LBS_ERR_ARG, "cum[0] must be 0");
  for (uint32_t l = 1; l <= max_len; ++l)
    if (cum[l] < cum[l - 1]) return fail(LBS_ERR_ARG, "cum must be non-decreasing");
  if (cum[max_len] == 0) return fail(LBS_ERR_ARG, "the dataset is empty");
  for (uint32_t s = 0; s < n_strata; ++s) {
    if (stratum_end[s] == 0 || stratum_end[s] > max_len || (s > 0 && stratum_end[s] <= stratum_end[s - 1]))
      return fail(LBS_ERR_ARG, "stratum_end must be increasing and lie in [1, max_len]");
  }
  if (stratum_end[n_strata - 1] != max_len) return fail(LBS_ERR_ARG, "the last stratum must end at max_len");
  lbs_dataset* ds = new lbs_dataset;
  *out = ds;  // from here on the caller's wrapper frees it on failure
  ds->max_len = max_len, ds->n_strata = n_strata;
  ds->cum.assign(cum, cum + max_len + 1);
  ds->stratum_end.assign(stratum_end, stratum_end + n_strata);
  if (device >= 0) {
    std::vector<uint32_t> guide(kWholeGuideSize + (size_t)n_strata * kGuideSize);
    ds->flagged = fill_guide<kWholeGuideBits>(guide.data(), ds->cum, 0, cum[max_len], 0);
    for (uint32_t s = 0; s < n_strata; ++s) {
      const uint32_t before = cum[s == 0 ? 0 : stratum_end[s - 1]];
      ds->flagged |= fill_guide<kGuideBits>(guide.data() + kWholeGuideSize + (size_t)s * kGuideSize, ds->cum, before,
                                            cum[stratum_end[s]] - before, s == 0 ? 0 : stratum_end[s - 1]);
    }
    int prev = -1;
    (void)hipGetDevice(&prev);
    hipError_t e = hipSetDevice(device);
    if (e == hipSuccess) ds->device = device;
    int n_cus = 0;
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e == hipSuccess) ds->n_cus = (uint32_t)std::max(n_cus, 1);
    if (e == hipSuccess) e = hipMalloc((void**)&ds->d_cum, (max_len + 1) * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemcpy(ds->d_cum, cum, (max_len + 1) * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc((void**)&ds->d_guide, guide.size() * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemcpy(ds->d_guide, guide.data(), guide.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (prev >= 0 && prev != device) (void)hipSetDevice(prev);
    if (e != hipSuccess) return fail(LBS_ERR_HIP, std::string("uploading the histogram: ") + hipGetErrorString(e));
  }
  return 0;
}

void lbs_dataset_destroy(lbs_dataset* ds) {
  if (!ds) return;
  if (ds->device >= 0 && (ds->d_cum || ds->d_guide)) {
    int prev = -1;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(ds->device);
    (void)hipDeviceSynchronize();
    if (ds->d_cum) (void)hipFree(ds->d_cum);
    if (ds->d_guide) (void)hipFree(ds->d_guide);
    if (prev >= 0 && prev != ds->device) (void)hipSetDevice(prev);
  }
  delete ds;
}

int lbs_dataset_create(lbs_dataset** out, int device, uint32_t max_len, const uint32_t* cum, uint32_t n_strata,
                       const uint32_t* stratum_end) {
  const int rc = no_throw([&] { return dataset_create(out, device, max_len, cum, n_strata, stratum_end); });
  if (rc != 0 && out && *out) {
    lbs_dataset_destroy(*out);
    *out = nullptr;
  }
  return rc;
}

// What a GPU's j-th draw comes from, stratum by stratum.
static int fill_slots(const lbs_dataset* ds, const lbs_run* run, Params* P) {
  uint32_t j = 0;
  for (uint32_t s = 0; s < ds->n_strata; ++s) {
    const uint32_t base = s == 0 ? 0 : ds->stratum_end[s - 1];
    const uint32_t lo = ds->cum[base], size = ds->cum[ds->stratum_end[s]] - lo;
    if (run->quota[s] && size == 0) return fail(LBS_ERR_ARG, "a stratum with a quota has no entries");
    if ((uint64_t)j + run->quota[s] > run->local_batch) return fail(LBS_ERR_ARG, "the quotas exceed local_batch");
    for (uint32_t q = 0; q < run->quota[s]; ++q, ++j)
      P->slot_lo[j] = lo, P->slot_size[j] = size, P->slot_guide[j] = s * kGuideSize, P->slot_base[j] = base;
  }
  if (j != run->local_batch) return fail(LBS_ERR_ARG, "the quotas must add up to local_batch");
  return 0;
}

// Packs the strata into at most two bins of 64 / gpus_per_node rows, largest quota first, each into the first bin with
// room; count = 0 if a stratum finds none (or gpus_per_node is not a power of two up to 16, or a GPU's tokens might not
// fit in 16 bits, which two nodes to a register need).
static Bins pack_bins(const lbs_dataset* ds, const lbs_run* run) {
  Bins L;
  memset(L.slot, kNoSlot, sizeof L.slot);
  L.count = 0, L.padded = 0;
  const uint32_t gpn = run->gpus_per_node;
  if (gpn == 0 || gpn > 16u || (gpn & (gpn - 1u)) != 0 || (uint64_t)run->local_batch * ds->max_len > 65534u) return L;
  const uint32_t rows = 64u / gpn;
  uint32_t used[2] = {0, 0};
  int bin_of[LBS_MAX_STRATA];
  uint32_t order[LBS_MAX_STRATA];  // by falling quota, equal ones in their order; on the stack: a call allocates nothing
  for (uint32_t s = 0; s < ds->n_strata; ++s) {
    uint32_t i = s;
    for (; i > 0 && run->quota[order[i - 1]] < run->quota[s]; --i) order[i] = order[i - 1];
    order[i] = s;
  }
  for (uint32_t i = 0; i < ds->n_strata; ++i) {
    const uint32_t s = order[i], q = run->quota[s];
    bin_of[s] = used[0] + q <= rows ? 0 : used[1] + q <= rows ? 1 : -1;
    if (bin_of[s] < 0) return L;
    used[bin_of[s]] += q;
  }
  uint32_t at[2] = {0, 0}, j = 0;
  for (uint32_t s = 0; s < ds->n_strata; ++s)
    for (uint32_t q = 0; q < run->quota[s]; ++q, ++j) L.slot[bin_of[s]][at[bin_of[s]]++] = (uint8_t)j;
  L.count = used[1] != 0 ? 2u : 1u;
  for (uint32_t b = 0; b < L.count; ++b)
    if (used[b] < rows) L.padded = 1;
  return L;
}

static uint32_t turn_of(uint32_t n_gpus) { return n_gpus > 1u ? (uint32_t)((1ull << 32) / n_gpus) + 1u : 0u; }

// One method of a run (run->method is not looked at).
static int simulate_one(const lbs_dataset* ds, const lbs_run* run, uint32_t method, uint32_t* trial_min, uint32_t* trial_max,
                        uint64_t* sums, void* stream) {
  if (!ds || !run) return fail(LBS_ERR_NULL, "dataset or run is NULL");
  if (method > LBS_GLOBAL) return fail(LBS_ERR_ARG, "unknown method");
  if (run->local_batch == 0 || run->n_gpus == 0) return fail(LBS_ERR_ARG, "local_batch and n_gpus must be positive");
  if (run->local_batch > LBS_MAX_LOCAL_BATCH) return fail(LBS_ERR_LIMIT, "local_batch exceeds LBS_MAX_LOCAL_BATCH");
  if ((uint64_t)run->n_gpus * run->local_batch >= (1ull << 31)) return fail(LBS_ERR_LIMIT, "n_gpus * local_batch must stay below 2^31");
  if (run->n_trials >= (1ull << 31)) return fail(LBS_ERR_LIMIT, "n_trials must stay below 2^31");
  const bool stratified = method == LBS_STRATIFIED || method == LBS_LOCAL_RASTER || method == LBS_LOCAL_SNAKE;
  const bool local = method == LBS_LOCAL_RASTER || method == LBS_LOCAL_SNAKE;
  Params P{};
  P.max_len = ds->max_len, P.local_batch = run->local_batch, P.gpus_per_node = run->gpus_per_node;
  P.n_gpus = run->n_gpus, P.snake = method == LBS_LOCAL_SNAKE, P.stratified = stratified;
  P.total = ds->cum[ds->max_len], P.seed = run->seed;
  P.guide_words = stratified ? ds->n_strata * kGuideSize : kWholeGuideSize;
  P.flagged = ds->flagged, P.turn = turn_of(run->n_gpus);
  if (stratified) {
    if (const int rc = fill_slots(ds, run, &P)) return rc;
  } else {
    for (uint32_t j = 0; j < run->local_batch; ++j) P.slot_lo[j] = 0, P.slot_size[j] = P.total, P.slot_guide[j] = 0, P.slot_base[j] = 0;
  }
  uint32_t pool = 0;
  if (local) {
    if (run->gpus_per_node == 0 || run->n_gpus % run->gpus_per_node) return fail(LBS_ERR_ARG, "n_gpus must be a multiple of gpus_per_node");
    if ((uint64_t)run->gpus_per_node * run->local_batch > LBS_MAX_NODE_POOL) return fail(LBS_ERR_LIMIT, "gpus_per_node * local_batch exceeds LBS_MAX_NODE_POOL");
    pool = run->gpus_per_node * run->local_batch;
  }
  if (!sums) return fail(LBS_ERR_NULL, "sums is NULL");
  if (ds->device < 0) return fail(LBS_ERR_HOST, "host-only dataset (device -1) cannot run kernels");
  int prev = -1;
  (void)hipGetDevice(&prev);
  if (prev != ds->device && hipSetDevice(ds->device) != hipSuccess) return fail(LBS_ERR_HIP, "hipSetDevice failed");
  hipStream_t s = (hipStream_t)stream;
  unsigned long long* ds_sums = reinterpret_cast<unsigned long long*>(sums);
  hipLaunchKernelGGL(k_lbs_clear, dim3(1), dim3(64), 0, s, ds_sums);
  hipError_t e = hipGetLastError();
  // dynamic LDS in words: histogram, guide tables, then the sorted pools (local) or the trial's histogram (global)
  const uint32_t tables = ds->max_len + 1u + P.guide_words;
  const bool spread = method == LBS_GLOBAL && run->n_gpus <= kMaxSpreadGpus;
  const size_t lds = sizeof(uint32_t) * (tables + (local ? kWaves * pool : method == LBS_GLOBAL ? ds->max_len + 1u + (spread ? run->n_gpus : 0u) : 0u));
  if (e == hipSuccess && run->n_trials > 0) {
    // trials cost the same, so a few workgroups per resident slot balance; each loops over its share of the trials
    const dim3 grid(trial_grid(run->n_trials, run->n_gpus, ds->n_cus)), block(kBlock);
    P.first_trial = run->first_trial, P.n_trials = (uint32_t)run->n_trials;
    const Bins L = local ? pack_bins(ds, run) : Bins{};
    const bool many_short = local && L.count == 1 && run->n_gpus / run->gpus_per_node <= kWaves &&
                            run->n_trials > (uint64_t)kBinsMostShortTrials * grid.x;
    if (local && L.count != 0 && !many_short) {
      hipLaunchKernelGGL(pick_bins<false>(L, run->gpus_per_node, run->n_gpus / run->gpus_per_node), grid, block, sizeof(uint32_t) * tables, s, P, L,
                         method, ds->d_cum, ds->d_guide, trial_min, trial_max, ds_sums);
    } else if (local) {
      const uint32_t gpn = run->gpus_per_node;
      const bool in_lanes = gpn <= 32 && (gpn & (gpn - 1u)) == 0;
      void (*kernel)(const Params, const uint32_t*, const uint32_t*, uint32_t*, uint32_t*, unsigned long long*) =
          pool <= 64    ? (in_lanes ? k_lbs_local<1, true> : k_lbs_local<1, false>)
          : pool <= 128 ? (in_lanes ? k_lbs_local<2, true> : k_lbs_local<2, false>)
          : pool <= 256 ? (in_lanes ? k_lbs_local<4, true> : k_lbs_local<4, false>)
          : pool <= 512 ? (in_lanes ? k_lbs_local<8, true> : k_lbs_local<8, false>)
                        : (in_lanes ? k_lbs_local<16, true> : k_lbs_local<16, false>);
      hipLaunchKernelGGL(kernel, grid, block, lds, s, P, ds->d_cum, ds->d_guide, trial_min, trial_max, ds_sums);
    } else if (method == LBS_GLOBAL) {
      hipLaunchKernelGGL(spread ? k_lbs_global<true> : k_lbs_global<false>, grid, block, lds, s, P, ds->d_cum, ds->d_guide, trial_min,
                         trial_max, ds_sums);
    } else {
      hipLaunchKernelGGL(stratified ? k_lbs_keep<kGuideBits> : k_lbs_keep<kWholeGuideBits>, grid, block, lds, s, P, ds->d_cum, ds->d_guide, trial_min, trial_max, ds_sums);
    }
    e = hipGetLastError();
  }
  if (prev >= 0 && prev != ds->device) (void)hipSetDevice(prev);
  if (e != hipSuccess) return fail(LBS_ERR_HIP, std::string("launching the simulation: ") + hipGetErrorString(e));
  return 0;
}

int lbs_simulate(const lbs_dataset* ds, const lbs_run* run, uint32_t* trial_min, uint32_t* trial_max, uint64_t* sums,
                 void* stream) {
  return no_throw([&] {
    if (!ds || !run) return fail(LBS_ERR_NULL, "dataset or run is NULL");
    return simulate_one(ds, run, run->method, trial_min, trial_max, sums, stream);
  });
}

static int simulate_all(const lbs_dataset* ds, const lbs_run* run, uint32_t* trial_min, uint32_t* trial_max, uint64_t* sums,
                        void* stream) {
  if (!ds || !run) return fail(LBS_ERR_NULL, "dataset or run is NULL");
  if (!sums) return fail(LBS_ERR_NULL, "sums is NULL");
  const uint32_t gpn = run->gpus_per_node, lb = run->local_batch, G = run->n_gpus;
  const uint32_t guide_words = kWholeGuideSize + ds->n_strata * kGuideSize;
  const size_t lds = sizeof(uint32_t) * (2u * (size_t)(ds->max_len + 1u) + guide_words + G);
  const bool one_pass = gpn != 0 && gpn <= 32 && (gpn & (gpn - 1u)) == 0 && lb != 0 && lb <= LBS_MAX_LOCAL_BATCH &&
                        (lb & (lb - 1u)) == 0 && G != 0 && G % gpn == 0 && G <= kMaxSpreadGpus && lds <= (60u << 10) &&
                        (uint64_t)gpn * lb <= LBS_MAX_NODE_POOL && ds->device >= 0 && run->n_trials > 0 &&
                        run->n_trials < (1ull << 31);
  if (!one_pass) {  // every other case, errors included: method by method
    for (uint32_t m = 0; m < kMethods; ++m) {
      const int rc = simulate_one(ds, run, m, trial_min ? trial_min + (size_t)m * run->n_trials : nullptr,
                                  trial_max ? trial_max + (size_t)m * run->n_trials : nullptr, sums + 2u * m, stream);
      if (rc != 0) return rc;
    }
    return 0;
  }
  Params P{};
  P.max_len = ds->max_len, P.local_batch = lb, P.gpus_per_node = gpn, P.n_gpus = G, P.stratified = 1;
  P.total = ds->cum[ds->max_len], P.seed = run->seed, P.first_trial = run->first_trial, P.n_trials = (uint32_t)run->n_trials;
  P.guide_words = guide_words;
  P.flagged = ds->flagged, P.turn = turn_of(G);
  if (const int rc = fill_slots(ds, run, &P)) return rc;
  int prev = -1;
  (void)hipGetDevice(&prev);
  if (prev != ds->device && hipSetDevice(ds->device) != hipSuccess) return fail(LBS_ERR_HIP, "hipSetDevice failed");
  hipStream_t s = (hipStream_t)stream;
  unsigned long long* ds_sums = reinterpret_cast<unsigned long long*>(sums);
  hipLaunchKernelGGL(k_lbs_clear_all, dim3(1), dim3(64), 0, s, ds_sums);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    const dim3 grid(trial_grid(run->n_trials, run->n_gpus, ds->n_cus)), block(kBlock);
    const uint32_t pool = gpn * lb;
    const Bins L = pack_bins(ds, run);
    void (*kernel)(const Params, const uint32_t*, const uint32_t*, uint32_t*, uint32_t*, unsigned long long*) =
        pool <= 64 ? k_lbs_all<1> : pool <= 128 ? k_lbs_all<2> : pool <= 256 ? k_lbs_all<4> : pool <= 512 ? k_lbs_all<8> : k_lbs_all<16>;
    if (L.count != 0)
      hipLaunchKernelGGL(pick_bins<true>(L, gpn, G / gpn), grid, block, lds, s, P, L, 0u, ds->d_cum,
                         ds->d_guide, trial_min, trial_max, ds_sums);
    else
      hipLaunchKernelGGL(kernel, grid, block, lds, s, P, ds->d_cum, ds->d_guide, trial_min, trial_max, ds_sums);
    e = hipGetLastError();
  }
  if (prev >= 0 && prev != ds->device) (void)hipSetDevice(prev);
  if (e != hipSuccess) return fail(LBS_ERR_HIP, std::string("launching the simulation: ") + hipGetErrorString(e));
  return 0;
}

int lbs_simulate_all(const lbs_dataset* ds, const lbs_run* run, uint32_t* trial_min, uint32_t* trial_max, uint64_t* sums,
                     void* stream) {
  return no_throw([&] { return simulate_all(ds, run, trial_min, trial_max, sums, stream); });
}

}  // extern "C"
