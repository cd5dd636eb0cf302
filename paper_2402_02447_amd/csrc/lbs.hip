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
//   LOCAL_*           : (k_lbs_bins, k_lbs_nodes, node sizes and quotas that fit) a wavefront owns a node or several;
//                       their strata, which are disjoint ranges of lengths and take whole rows of the sorted pool,
//                       are packed into bins of 64 entries, two bins to a register as 16-bit halves, and sorted there;
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
  bool whole_first = false;     // k_lbs_nodes with the whole dataset's table has no LDS in front of that table
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

// Guide entries.  A draw's upper BITS bits select the cell, the draw is added to the entry (modulo 2^32), and the sum's
// upper BITS bits are the length (counted from the length below the range's first one): an entry is (l - cell) * 2^(32 - BITS)
// for a cell that selects l only, and 2^(32 - BITS) - from more for one that selects l + 1 from the lower bits `from` on.
// Cells that have to be searched have kFlagged and more where the others have l * 2^(32 - BITS): bits 0 .. 9 hold the
// smallest length minus one, bits 10 .. 19 how far the largest one lies above it.  (An addition and a shift, which issue in
// two cycles each here; comparing with a threshold instead takes three instructions of four cycles.)
template <uint32_t BITS>
constexpr uint32_t kFlagged = ((1u << BITS) - 1u) << (32u - BITS);

// The draw with generator state z: the upper half of the generator's output.
__device__ __forceinline__ uint32_t drawn(uint64_t z) { return (uint32_t)(mix(z) >> 32); }

// The same in fewer, longer instructions: a * b + c on 64 bits costs what a 32-bit multiplication does, but the compiler takes it
// apart where only the sum's lower half is used.  61 instead of 66 cycles of issue a draw, for kernels that are bound by that (five methods at
// 1 024 GPUs 463 -> 453 us, snake 370 -> 343); those that wait rather than issue lose by the longer chain (one node of 8, batch 8:
// 1827 -> 2100).
__device__ __forceinline__ uint64_t mad64(uint32_t a, uint32_t b, uint64_t c) {
  uint64_t d, carry;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(d), "=s"(carry) : "v"(a), "s"(b), "v"(c));
  return d;
}
__device__ __forceinline__ uint32_t drawn_dense(uint64_t z) {
  constexpr uint32_t A = 0xBF58476Du, B = 0x1CE4E5B9u, C = 0x94D049BBu, D = 0x133111EBu;  // mix's multipliers, halves
  z ^= z >> 30;
  const uint64_t y = (uint64_t)(uint32_t)z * B;
  const uint64_t cross = mad64((uint32_t)(z >> 32), B, (uint64_t)(uint32_t)z * A);
  z = ((uint64_t)((uint32_t)(y >> 32) + (uint32_t)cross) << 32) | (uint32_t)y;
  z ^= z >> 27;
  uint32_t any;
  asm("" : "=v"(any));  // of the sums that follow only the lower words are used
  const uint64_t carried = (uint64_t)any << 32 | __umulhi((uint32_t)z, D);
  const uint32_t u = (uint32_t)mad64((uint32_t)(z >> 32), D, mad64((uint32_t)z, C, carried));
  return u ^ (u >> 31);
}

// Length selected by draw u; `guide` is its range's table, `base` the length below the range's first one.  FLAGGED: some
// entry may be flagged; `range` then says which dataset entries the draw is from.  WHOLE_ENTRY: the cell's first draw has
// been added to the entries (load_tables).
template <uint32_t BITS, bool FLAGGED, bool WHOLE_ENTRY = false, typename F>
__device__ __forceinline__ uint32_t length_of(const uint32_t* s_cum, const uint32_t* guide, uint32_t u, uint32_t base, F range) {
  constexpr uint32_t kLow = (1u << (32u - BITS)) - 1u;
  const uint32_t at = guide[u >> (32u - BITS)];
  uint32_t l = base + ((at + (WHOLE_ENTRY ? u & kLow : u)) >> (32u - BITS));
  if constexpr (FLAGGED) {
    const uint32_t e = WHOLE_ENTRY ? at : at + (u & ~kLow);
    if (e >= kFlagged<BITS>) {
      const uint32_t lo = (e & 1023u) + 1u;
      uint32_t before, size;
      range(before, size);
      l = first_above(s_cum, lo, lo + ((e >> 10) & 1023u), before + __umulhi(u, size));
    }
  }
  return l;
}

// Histogram and guide tables into LDS; returns where the guide tables start.  BITS != 0: with each cell's first draw (its
// place in its table of 2^BITS cells) added to its entry.
template <uint32_t BITS = 0>
__device__ __forceinline__ uint32_t* load_tables(uint32_t* s_dyn, const Params& P, const uint32_t* __restrict__ cum,
                                                 const uint32_t* __restrict__ guide) {
  uint32_t* s_guide = s_dyn + P.max_len + 1u;
  for (uint32_t i = threadIdx.x; i <= P.max_len; i += kBlock) s_dyn[i] = cum[i];
  const uint32_t* src = guide + (P.stratified ? kWholeGuideSize : 0u);  // the whole dataset's table comes first
  for (uint32_t i = threadIdx.x; i < P.guide_words; i += kBlock) s_guide[i] = src[i] + (BITS != 0 ? i << ((32u - BITS) & 31u) : 0u);
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
// The cells' first draws are added to the entries while they are loaded, which the other kernels leave out: there the sum with the
// whole draw is an instruction less, here one that takes the draw's last xor and the sum together, after the lookup, and is 1 % slower
// (4 to 5 % in places: batch 32, 14 nodes of 16, 41 852 trials, 240 us against 230).
template <uint32_t BITS>
__global__ __launch_bounds__(kBlock) void k_lbs_keep(const Params P, const uint32_t* __restrict__ cum,
                                                      const uint32_t* __restrict__ guide, uint32_t* trial_min,
                                                      uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, guide tables
  __shared__ Finish s_finish;
  const uint32_t* s_guide = load_tables<BITS>(s_dyn, P, cum, guide);
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
          tokens += length_of<BITS, decltype(fl)::value, true>(
              s_dyn, s_guide + P.slot_guide[j], drawn(z), P.slot_base[j],
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
            v[e] = i < pool ? length_of<kGuideBits, decltype(fl)::value>(
                                  s_dyn, s_guide + goff[e], drawn(z_node + i * kGamma), base_len[e],
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
        atomicAdd(&s_cnt[length_of<kWholeGuideBits, decltype(fl)::value>(
                      s_dyn, s_guide, drawn(z), 0u, [&](uint32_t& before, uint32_t& size) { before = 0u, size = P.total; })],
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
// Draw number k of a run does not depend on the method, and it belongs to the same GPU and the same one of its local_batch
// sequences in all of them: NONE and GLOBAL look it up in the whole dataset, STRATIFIED and the LOCAL methods in the
// sequence's stratum.  So one generator output (most of what a draw costs: two 64-bit multiplications) serves both.
// A wavefront takes a node (or several), makes its draws, counts the lengths from the whole dataset for the counting
// sort (GLOBAL, as in k_lbs_global<true>), adds up each GPU's own lengths of either kind (NONE, STRATIFIED), sorts the
// stratified ones and deals twice (LOCAL_RASTER, LOCAL_SNAKE).
constexpr uint32_t kMethods = 5;

// A trial's draws from the whole dataset are counted in s_cnt between these two.  All threads of the workgroup call both, with
// a barrier after the first and one before the second; s_cnt, s_gpu, *s_base and s_scan are theirs until the next barrier
// of the caller.
__device__ __forceinline__ void whole_clear(const Params& P, uint32_t* s_cnt, uint32_t* s_gpu, uint32_t* s_base) {
  for (uint32_t i = threadIdx.x; i <= P.max_len; i += kBlock) s_cnt[i] = 0u;
  for (uint32_t i = threadIdx.x; i < P.n_gpus; i += kBlock) s_gpu[i] = 0u;
  if (threadIdx.x == 0) *s_base = 0u;
}

// GLOBAL: the counted lengths dealt over all GPUs as in k_lbs_global<true>; smallest and largest sum of this thread's GPUs.
__device__ __forceinline__ void whole_deal(const Params& P, const uint32_t* s_cnt, uint32_t* s_gpu, uint32_t* s_base,
                                           uint32_t (*s_scan)[kWaves], uint32_t& glob_lo, uint32_t& glob_hi) {
  const uint32_t tid = threadIdx.x;
  const uint32_t per = (P.max_len + 1u + kBlock - 1u) / kBlock;
  const uint32_t a = tid * per, b = min(a + per, P.max_len + 1u);
  const uint32_t per_gpu = (P.n_gpus + kBlock - 1u) / kBlock;
  const uint32_t ga = min(tid * per_gpu, P.n_gpus), gb = min(ga + per_gpu, P.n_gpus);
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

// Minima and maxima of a trial, one for every 32 lanes.  BUFFERS == 2: in turn by the parity of the workgroup's trial count; trials of all five methods
// have a barrier between one's reading and the next one's filing, and need one.  Kept small: with 8 000 simulated GPUs 960 bytes more made three
// workgroups a compute unit two (12 000 trials of 250 nodes of 32, batch 4: 1 891 -> 2 326 us).
constexpr uint32_t kRows = 2u * kWaves;
template <uint32_t BUFFERS>
struct FinishAll {
  uint32_t lo[BUFFERS][kMethods][kRows], hi[BUFFERS][kMethods][kRows];
};
static_assert(sizeof(FinishAll<1>) <= 320);

// Minimum and maximum over each row of 16 lanes, in all of its lanes.
__device__ __forceinline__ void row_min_max(uint32_t& lo, uint32_t& hi) {
  const auto step = [&](auto rotate) {
    lo = min(lo, (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, decltype(rotate)::value, 0xf, 0xf, true));
    hi = max(hi, (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, decltype(rotate)::value, 0xf, 0xf, true));
  };
  step(std::integral_constant<int, 0x128>{}), step(std::integral_constant<int, 0x124>{});
  step(std::integral_constant<int, 0x122>{}), step(std::integral_constant<int, 0x121>{});
}

// Files the minimum and maximum that the wavefront's lanes have seen of method q.
template <uint32_t BUFFERS>
__device__ __forceinline__ void file_min_max(FinishAll<BUFFERS>& fin, uint32_t buf, uint32_t q, uint32_t lo, uint32_t hi) {
  row_min_max(lo, hi);
  // rows 0 and 2 to rows 1 and 3
  lo = min(lo, (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, 0x142, 0xa, 0xf, false));
  hi = max(hi, (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, 0x142, 0xa, 0xf, false));
  const uint32_t tid = threadIdx.x;
  if ((tid & 31u) == 16u) fin.lo[buf][q][tid >> 5] = lo, fin.hi[buf][q][tid >> 5] = hi;
}

// A trial's results from what has been filed in the first ROWS places: thread 2 q stores method q's minimum, thread 2 q + 1 its
// maximum, and adds it to the workgroup's sums.  all: the five methods, else `method` alone.
template <uint32_t ROWS = kRows, uint32_t BUFFERS>
__device__ __forceinline__ void finish_methods(const Params& P, const FinishAll<BUFFERS>& fin, unsigned long long* s_sum, uint32_t buf, uint32_t t,
                                               bool all, uint32_t method, uint32_t* trial_min, uint32_t* trial_max) {
  const uint32_t tid = threadIdx.x, m = tid >> 1;
  if (tid >= 2u * kMethods || (!all && m != method)) return;
  const size_t at = all ? (size_t)m * P.n_trials + t : t;
  uint32_t x;
  if (tid & 1u) {
    x = 0u;
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r) x = max(x, fin.hi[buf][m][r]);
    if (trial_max) trial_max[at] = x;
  } else {
    x = 0xffffffffu;
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r) x = min(x, fin.lo[buf][m][r]);
    if (trial_min) trial_min[at] = x;
  }
  s_sum[tid] += x;
}

// A wavefront per node, whose pool lies in registers (entry i in register i / 64 of lane i % 64) and is sorted as in
// k_lbs_local<E, true>; a GPU's own draws are local_batch consecutive entries, added up by a butterfly over the low lane
// bits.  Needs gpus_per_node and local_batch to be powers of two (<= 32 and <= 64).
template <int E>
__global__ __launch_bounds__(kBlock, E <= 2 ? 6 : E == 4 ? 4 : E == 8 ? 3 : 2) void k_lbs_all(const Params P, const uint32_t* __restrict__ cum,
                                                     const uint32_t* __restrict__ guide, uint32_t* trial_min,
                                                     uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, all guide tables, the trial's own histogram, one word per GPU
  __shared__ uint32_t s_scan[2][kWaves];
  __shared__ uint32_t s_base;
  __shared__ FinishAll<1> s_fin;
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
  const bool halves = P.local_batch * P.max_len < 65536u;

  for (uint32_t t = blockIdx.x; t < P.n_trials; t += gridDim.x) {
    uint32_t lo[kMethods], hi[kMethods];
#pragma unroll
    for (uint32_t q = 0; q < kMethods; ++q) lo[q] = 0xffffffffu, hi[q] = 0u;
    const uint64_t k_trial = (P.first_trial + t) * (uint64_t)pool_all;  // the trial's first draw
    whole_clear(P, s_cnt, s_gpu, &s_base);
    __syncthreads();
    for (uint32_t node = wave; node < n_nodes; node += kWaves) {
      const uint64_t z_node = state(P.seed, k_trial + (uint64_t)node * pool);
      uint32_t v[E];
      const auto draws = [&](auto fl) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const uint32_t i = (uint32_t)e * 64u + lane;
          const bool real = i < pool;
          uint32_t w = 0u;
          v[e] = 0xffffffffu;
          if (real) {
            const uint32_t u = drawn(z_node + i * kGamma);
            v[e] = length_of<kGuideBits, decltype(fl)::value>(s_dyn, s_strata + goff[e], u, base_len[e],
                                                              [&](uint32_t& before, uint32_t& size) {
                                                                before = P.slot_lo[i % P.local_batch], size = P.slot_size[i % P.local_batch];
                                                              });
            w = length_of<kWholeGuideBits, decltype(fl)::value>(
                s_dyn, s_whole, u, 0u, [&](uint32_t& before, uint32_t& size) { before = 0u, size = P.total; });
            atomicAdd(&s_cnt[w], 1u);
          }
          // a GPU's own draws; both kinds in one word where the sums fit in 16 bits
          const auto own = [&](uint32_t q, uint32_t tokens) {
            if (real) lo[q] = min(lo[q], tokens), hi[q] = max(hi[q], tokens);
          };
          if (halves) {
            const uint32_t both = butterfly_sum(real ? v[e] | w << 16 : 0u, 0u, batch_bit);
            own(LBS_STRATIFIED, both & 0xffffu), own(LBS_NONE, both >> 16);
          } else {
            own(LBS_STRATIFIED, butterfly_sum(real ? v[e] : 0u, 0u, batch_bit));
            own(LBS_NONE, butterfly_sum(w, 0u, batch_bit));
          }
        }
      };
      if (P.flagged != 0u) draws(std::true_type{});
      else draws(std::false_type{});
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
    __syncthreads();
    whole_deal(P, s_cnt, s_gpu, &s_base, s_scan, lo[LBS_GLOBAL], hi[LBS_GLOBAL]);
    // ---- the trial's five results
#pragma unroll
    for (uint32_t q = 0; q < kMethods; ++q) file_min_max(s_fin, 0u, q, lo[q], hi[q]);
    __syncthreads();  // also: this trial's last reads of s_cnt and s_gpu lie before the next trial's clearing
    finish_methods(P, s_fin, s_sum, 0u, t, true, 0u, trial_min, trial_max);
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
//   Workgroups a compute unit: six, but for all five methods with eight columns a lane five (99 registers at four of them; 12 000 trials of 64 nodes of 8,
// cells to be searched: at four 383 us, five 347, six 341; 30 nodes in one bin 191, 172, 175).
//   Measured (20 000 trials of 1 024 GPUs x 16, nodes of 8): snake alone 420 us (k_lbs_local 637), nodes of 4: 476 (1168 all five).  Bins that
// are full go by k_lbs_nodes where there are many nodes; those with padding, datasets with flagged entries, other node sizes and few nodes
// stay here.  Five methods, 24 414 trials of 128 nodes of 8: one node at a time 796 us, columns in registers 613 (792 before the two kinds of
// draws shared the generator's outputs); 390 625 trials of 8 nodes: 1 302 and 1 965 (1 910).
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
__global__ __launch_bounds__(kBlock, WHOLE && LG == 3 ? 5 : 6) void k_lbs_bins(const Params P, const Bins L, const uint32_t method,
                                                         const uint32_t* __restrict__ cum, const uint32_t* __restrict__ guide,
                                                         uint32_t* trial_min, uint32_t* trial_max, unsigned long long* sums) {
  extern __shared__ uint32_t s_dyn[];  // histogram, guide tables; WHOLE: the trial's own histogram, one word per GPU
  __shared__ uint32_t s_scan[2][kWaves];
  __shared__ uint32_t s_base;
  __shared__ FinishAll<WHOLE ? 1 : 2> s_fin;
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
    const uint32_t buf = WHOLE ? 0u : round & 1u;
    const uint64_t k_trial = (P.first_trial + t) * (uint64_t)pool_all;
    if (WHOLE) {
      whole_clear(P, s_cnt, s_gpu, &s_base);
      __syncthreads();
    }
    // Running minima and maxima: LG > 0, of own, raster, snake and (WHOLE) what the GPUs draw from the whole dataset in turn;
    // LG == 0, one for all, told apart by the lane.  BINS == 1: 16-bit halves.
    constexpr int S = WHOLE ? 4 : 3, M = LG > 0 ? S : 1;
    uint32_t lo[M], hi[M];
#pragma unroll
    for (int m = 0; m < M; ++m) lo[m] = 0xffffffffu, hi[m] = 0u;
    for (uint32_t first = wave * kNodes; first < n_nodes; first += kWaves * kNodes) {
      const uint64_t z0 = state(P.seed, k_trial + (uint64_t)first * pool);
      uint32_t v[R], whole[R];
      const auto draws = [&](auto fl) {
#pragma unroll
        for (int c = 0; c < R; ++c) {
          uint32_t d[2], w[2] = {};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t u = drawn(z0 + (uint64_t)c * next_column + step[h]);
            d[h] = length_of<kGuideBits, decltype(fl)::value>(
                s_dyn, s_strata + goff[h], u, base_len[h],
                [&](uint32_t& before, uint32_t& size) { before = P.slot_lo[slot[h]], size = P.slot_size[slot[h]]; });
            if (WHOLE) {
              w[h] = length_of<kWholeGuideBits, decltype(fl)::value>(
                  s_dyn, s_whole, u, 0u, [&](uint32_t& before, uint32_t& size) { before = 0u, size = P.total; });
              // padding and nodes that are not there count for nothing
              const uint32_t node = LG == 0 ? first + (BINS == 2 ? 0u : (uint32_t)h) : first + (BINS == 2 ? group : group * 2u + (uint32_t)h);
              if (node < n_nodes && (real & (h == 0 ? 0xffffu : 0xffff0000u)) != 0u) atomicAdd(&s_cnt[w[h]], 1u);
            }
          }
          v[c] = d[0] | (d[1] << 16), whole[c] = w[0] | (w[1] << 16);
        }
      };
      if (P.flagged != 0u) draws(std::true_type{});
      else draws(std::false_type{});
      if (first + kNodes > n_nodes) {  // the last nodes: others take the place of those that are not there
        const uint32_t node = first + (BINS == 2 ? group : group * 2u);
        // BINS == 1: a second node that is not there repeats the first; a whole group that is not there is left out below
        if (BINS == 1 && node + 1u >= n_nodes) {
#pragma unroll
          for (int c = 0; c < R; ++c) v[c] = (v[c] & 0xffffu) | (v[c] << 16), whole[c] = (whole[c] & 0xffffu) | (whole[c] << 16);
        }
      }
      const bool there = LG == 0 || first + (BINS == 2 ? group : group * 2u) < n_nodes;
      uint32_t own[R];
#pragma unroll
      for (int c = 0; c < R; ++c) own[c] = v[c];
      if (L.padded != 0u) {
        // 0xffff sorts behind every length, into the bin's last rows: again the padded ones
#pragma unroll
        for (int c = 0; c < R; ++c) own[c] &= real, whole[c] &= real, v[c] |= ~real;
      }
      uint32_t sum[4] = {};
      if constexpr (LG > 0) {
        sum[0] = column_sums<LG>(own, bit);
        if (WHOLE) sum[3] = column_sums<LG>(whole, bit);
      } else {
        sum[0] = own[0], sum[3] = whole[0];
      }
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
        for (int m = 0; m < S; ++m) sum[m] = (sum[m] & 0xffffu) + (sum[m] >> 16);
      }
      if constexpr (LG > 0) {
        if (there) {
#pragma unroll
          for (int m = 0; m < S; ++m) {
            lo[m] = BINS == 2 ? min(lo[m], sum[m]) : min_halves(lo[m], sum[m]);
            hi[m] = BINS == 2 ? max(hi[m], sum[m]) : max_halves(hi[m], sum[m]);
          }
        }
      } else {
        // sums over the rows of 16 lanes: row 0 ends up with `own`, row 2 with `raster`, row 1 with `snake`, row 3 with it or
        // (WHOLE) with the draws from the whole dataset
        const auto p = __builtin_amdgcn_permlane32_swap(sum[0], sum[1], false, false);
        const auto q = __builtin_amdgcn_permlane32_swap(sum[2], WHOLE ? sum[3] : sum[2], false, false);
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
      if (LG > 0) {
        file_min_max(s_fin, buf, m == 0 ? LBS_STRATIFIED : m == 1 ? LBS_LOCAL_RASTER : m == 2 ? LBS_LOCAL_SNAKE : LBS_NONE, lo[m], hi[m]);
      } else {  // a row of lanes stands for the whole wavefront
        row_min_max(lo[m], hi[m]);
        const uint32_t which = lane >> 4, i = lane & 15u;
        const uint32_t q = which == 0u ? LBS_STRATIFIED : which == 1u ? LBS_LOCAL_SNAKE : which == 2u ? LBS_LOCAL_RASTER : LBS_NONE;
        // One method alone: one place a wavefront, as a trial of a node or two is hardly longer than its end (one node of 8, batch 16, 400 000
        // trials: 276 us, with four places a wavefront 293).
        if (WHOLE ? i < 2u : i == 0u && which < 3u) {
          const uint32_t at = WHOLE ? wave * 2u + i : wave;
          s_fin.lo[buf][q][at] = lo[m], s_fin.hi[buf][q][at] = hi[m];
        }
      }
    }
    if (WHOLE) {
      uint32_t glob_lo = 0xffffffffu, glob_hi = 0u;
      __syncthreads();
      whole_deal(P, s_cnt, s_gpu, &s_base, s_scan, glob_lo, glob_hi);
      file_min_max(s_fin, buf, LBS_GLOBAL, glob_lo, glob_hi);
    }
    __syncthreads();  // also: this trial's last reads of s_cnt and s_gpu lie before the next trial's clearing
    finish_methods<LG == 0 && !WHOLE ? kWaves : kRows>(P, s_fin, s_sum, buf, t, WHOLE, method, trial_min, trial_max);
  }
  if (tid < 2u * kMethods && (WHOLE || (tid >> 1) == method)) atomicAdd(&sums[WHOLE ? tid : (tid & 1u)], s_sum[tid]);
}

// ---- node-local methods with the strata in full bins, most of the sort inside a lane --------------------
// As k_lbs_bins, for nodes of 2^CB GPUs (CB 2 or 3) whose bins are full and datasets without flagged guide entries.  A
// node (BINS == 2) or a pair of nodes (BINS == 1) lies in 64 / R lanes of R = 2^LG registers.  The more registers, the fewer
// of the 21 stages cross lanes (R = 8: 6, 16: 3, 32: 1), and what happens inside a lane can use Batcher's odd-even merge
// sort (63 comparisons for 16 values instead of the bitonic network's 80).
//   Before the sort any entry of a bin may lie anywhere in it, so a lane draws all rows of a few columns, i.e. everything
// that 2^(CB + LG - 6) GPUs draw: which stratum an entry is from is then the same in all lanes (scalar registers, not vector
// ones), and what a GPU draws itself adds up within the lane.
//   After the sort lanes with an odd number hold complements in falling order (sort_columns): entry (row, column) of such a lane
// lies where the other lanes have the mirrored row and column, so that of two neighbours each keeps the first half of its
// column sums and gets the other's second half, backwards, added to it.
//   Bound: vector issue (0.87 of the time; a wavefront's 32 nodes cost 8 800 cycles, of which the generator takes 3 900, the look-ups
// 2 100 and the sort 2 600).  100 000 trials of 1 024 GPUs x 16, nodes of 8, all five methods: 3 093 us before (every generator output made twice,
// 8 registers), 2 240 with 8 registers, 2 006 with 16, 1 769 with 32; snake alone, 24 414 trials, 514 -> 341.  Which number of
// registers, and where one node at a time is better, Cost says.
//   The registers that so many workgroups a compute unit leave (96 and 80) are a few too few for some: <5, 3, 2, true>, whose time is above, spills
// four a lane, <5, 3, 1, true> ten, <5, 3, 1, false> three, <5, 2, 2, true> and <4, 3, 1, true> two, the others none.
template <int LG, int CB, int BINS>
constexpr uint32_t kNodesAtOnce = (1u << LG) * (BINS == 2 ? 1u : 2u);  // nodes a wavefront takes at a time

constexpr uint32_t kCountWords = 1028;  // a trial's histogram: lengths 0 .. LBS_MAX_LEN
static_assert(kCountWords > LBS_MAX_LEN && kCountWords % 4 == 0);
typedef const __attribute__((address_space(3))) uint32_t lds_word;
template <bool WHOLE>
struct NodesShared {
  unsigned long long sum[2u * kMethods];
  FinishAll<WHOLE ? 1 : 2> fin;
  uint32_t scan[2][kWaves];
  uint32_t base, unused;
};
static_assert(sizeof(NodesShared<false>) % 8 == 0 && sizeof(NodesShared<true>) % 8 == 0);

struct Rows {  // row r of bin h: base | stratum << 16 | slot << 24 (see Bins)
  uint32_t row[2][16];
  uint32_t odd[2];  // bit r: the slot of row r is odd
};

__device__ __forceinline__ void order_halves(uint32_t& a, uint32_t& b) {
  const uint32_t x = min_halves(a, b), y = max_halves(a, b);
  a = x, b = y;
}

// Sorts the halves of every group of 2^(6 - LG) lanes as sort_halves<LG> does, except that lanes with an odd number end up with
// complements, their registers in reverse order.  In: values as they are, in any order.
//   Runs that are merged next run in opposite directions, and as what a run's partner does in the merge after that is free, the
// directions are taken such that the first stage of a merge finds every lane in the form that it needs.
template <int LG>
__device__ __forceinline__ void sort_columns(uint32_t (&v)[1 << LG], const uint32_t (&bit)[6]) {
  constexpr int R = 1 << LG;
  uint32_t falls[7];  // falls[lk]: lanes whose run of 2^lk entries is sorted in falling order
  falls[6] = 0u;
#pragma unroll
  for (int lk = 5; lk >= LG; --lk) falls[lk] = falls[lk + 1] ^ bit[lk - LG];
#pragma unroll
  for (int c = 0; c < R; ++c) v[c] ^= falls[LG];
  // odd-even merge sort of the registers: lanes that hold complements sort in falling order
#pragma unroll
  for (int p = 1; p < R; p <<= 1) {
#pragma unroll
    for (int k = p; k >= 1; k >>= 1) {
#pragma unroll
      for (int j = k % p; j + k < R; j += 2 * k) {
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < R && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order_halves(v[i + j], v[i + j + k]);
      }
    }
  }
#pragma unroll
  for (int lk = LG + 1; lk <= 6; ++lk) {  // bitonic merges
#pragma unroll
    for (int lj = lk - 1; lj >= LG; --lj) {  // across lanes: see sort_halves
#pragma unroll
      for (int c = 0; c < R; ++c) v[c] = min_halves(v[c], ~partner_of(v[c], lj - LG));
      // the form of the next stage; the last merge ends as it is
      const uint32_t change = lj > LG ? bit[lj - LG] ^ bit[lj - 1 - LG] : lk < 6 ? bit[0] : 0u;
      if (lj > LG || lk < 6) {
#pragma unroll
        for (int c = 0; c < R; ++c) v[c] ^= change;
      }
    }
#pragma unroll
    for (int lj = LG - 1; lj >= 0; --lj) {
#pragma unroll
      for (int c = 0; c < R; ++c)
        if (!(c & (1 << lj))) order_halves(v[c], v[c | (1 << lj)]);
    }
  }
}

template <int LG, int CB, int BINS, bool WHOLE>
__global__ __launch_bounds__(kBlock, LG == 5 ? 5 : 6) void k_lbs_nodes(
    const Params P, const Rows L, const uint32_t method, const uint32_t* __restrict__ guide, uint32_t* trial_min, uint32_t* trial_max,
    unsigned long long* sums) {
  constexpr uint32_t R = 1u << LG, C = 1u << CB, LANES = 64u >> LG, ROWS = 64u >> CB;
  constexpr uint32_t CPL = C / LANES;  // columns a lane draws
  constexpr uint32_t RPL = R / C;      // rows a lane holds once sorted
  static_assert(CPL >= 1 && RPL >= 1 && CPL * ROWS == R && RPL * LANES == ROWS && ROWS <= 16);
  // (WHOLE) the whole dataset's guide table and the trial's own histogram; the strata's tables, NodesShared, a word per GPU.  The kernel
  // has no static LDS, so that this is address 0 and a draw's upper bits are the address of its entry in the first table (an
  // addition of the array's address, which the compiler does not fold away, is a fortieth of a draw).  whole_tables_first() looks
  // whether that is so; where it is not, the kernel is not launched.
  extern __shared__ uint32_t s_dyn[];
  constexpr uint32_t kCnt = kWholeGuideSize, kStrata = WHOLE ? kCnt + kCountWords : 0u;
  uint32_t* s_strata = s_dyn + kStrata;
  uint32_t* s_cnt = s_dyn + kCnt;
  const uint32_t strata_words = P.guide_words - (WHOLE ? kWholeGuideSize : 0u);
  NodesShared<WHOLE>& sh = *reinterpret_cast<NodesShared<WHOLE>*>(s_strata + strata_words);
  uint32_t* s_gpu = s_strata + strata_words + sizeof(NodesShared<WHOLE>) / sizeof(uint32_t);
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < 2u * kMethods) sh.sum[tid] = 0ull;
  if (WHOLE)
    for (uint32_t i = tid; i < kWholeGuideSize; i += kBlock) s_dyn[i] = guide[i];
  for (uint32_t i = tid; i < strata_words; i += kBlock) s_strata[i] = guide[kWholeGuideSize + i];
  __syncthreads();

  const uint32_t pool_all = P.n_gpus * P.local_batch;
  const uint32_t n_nodes = P.n_gpus / C;
  const uint32_t pool = C * P.local_batch;
  const uint32_t group = lane / LANES, part = lane % LANES;
  uint32_t bit[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) bit[q] = 0u - ((lane >> q) & 1u);
  uint32_t odd[RPL];  // halves of odd rows among those this lane holds once sorted
#pragma unroll
  for (uint32_t r = 0; r < RPL; ++r) {
    const uint32_t row = part * RPL + ((part & 1u) ? RPL - 1u - r : r);
    odd[r] = (((L.odd[0] >> row) & 1u) ? 0xffffu : 0u) | (((L.odd[BINS == 2 ? 1 : 0] >> row) & 1u) ? 0xffff0000u : 0u);
  }
  const uint32_t uncomplement = bit[0] & (1u - RPL);  // a sum of RPL complements is that many less one, complemented

  uint32_t rows[BINS == 2 ? 2 : 1][ROWS];
#pragma unroll
  for (uint32_t h = 0; h < (BINS == 2 ? 2u : 1u); ++h)
#pragma unroll
    for (uint32_t r = 0; r < ROWS; ++r) rows[h][r] = L.row[h][r];

  for (uint32_t t = blockIdx.x, round = 0; t < P.n_trials; t += gridDim.x, ++round) {
    const uint32_t buf = WHOLE ? 0u : round & 1u;
    const uint64_t k_trial = (P.first_trial + t) * (uint64_t)pool_all;
    if (WHOLE) {
      whole_clear(P, s_cnt, s_gpu, &sh.base);
      __syncthreads();
    }
    const uint64_t z_trial = state(P.seed, k_trial);
    uint32_t lo[4], hi[4];  // none, own, raster, snake; BINS == 1: the last three are 16-bit halves
#pragma unroll
    for (int m = 0; m < 4; ++m) lo[m] = 0xffffffffu, hi[m] = 0u;
    // `absent` (all ones where there is no node) leaves a minimum as it is, as zero leaves a maximum
    const auto note = [&](int m, uint32_t x, uint32_t absent) { lo[m] = min(lo[m], x | absent), hi[m] = max(hi[m], x & ~absent); };
    const auto note_halves = [&](int m, uint32_t x, uint32_t absent) {
      if (BINS == 2) note(m, (x & 0xffffu) + (x >> 16), absent);
      else lo[m] = min_halves(lo[m], x | absent), hi[m] = max_halves(hi[m], x & ~absent);
    };
    for (uint32_t first = wave * kNodesAtOnce<LG, CB, BINS>; first < n_nodes; first += kWaves * kNodesAtOnce<LG, CB, BINS>) {
      // A group whose nodes are not there makes somebody else's draws (the same ones in several lanes would be counted one after
      // the other), which count for nothing; the second of a pair that is not there repeats the first.
      const bool there = first + (BINS == 2 ? group : group * 2u) < n_nodes;
      const uint32_t absent = there ? 0u : 0xffffffffu;
      uint64_t z[BINS == 2 ? 1 : 2];
      uint32_t one[BINS == 2 ? 1 : 2];
#pragma unroll
      for (uint32_t h = 0; h < (BINS == 2 ? 1u : 2u); ++h) {
        const uint32_t node = first + (BINS == 2 ? group : group * 2u + h);
        one[h] = node < n_nodes ? 1u : 0u;
        const uint32_t whose = BINS == 1 && h == 1 && there && node >= n_nodes ? node - 1u : node;
        z[h] = z_trial + (uint64_t)(whose * pool + part * CPL * P.local_batch) * kGamma;
      }
      uint32_t v[R], own[CPL] = {}, none[BINS == 2 ? 1 : 2][CPL] = {};
#pragma unroll
      for (uint32_t r = 0; r < ROWS; ++r) {
        uint32_t info[2], u[2][CPL], w[2][CPL], d[2][CPL];
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
          info[h] = rows[BINS == 2 ? h : 0][r];
          asm volatile("" : "+s"(info[h]));  // what follows from it is recomputed here: kept from round to round, it would fill the scalar registers
#pragma unroll
          for (uint32_t c = 0; c < CPL; ++c) {
            uint64_t ahead = (uint64_t)(c * P.local_batch + (info[h] >> 24)) * kGamma;
            asm("" : "+s"(ahead));  // the product is the scalar unit's
            u[h][c] = LG >= 4 ? drawn_dense(z[BINS == 2 ? 0 : h] + ahead) : drawn(z[BINS == 2 ? 0 : h] + ahead);
          }
        }
        // every table lookup of the row is under way before the first one is needed
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
#pragma unroll
          for (uint32_t c = 0; c < CPL; ++c) {
            d[h][c] = s_strata[((info[h] >> 16) & 255u) * kGuideSize + (u[h][c] >> (32u - kGuideBits))];
            if (WHOLE) w[h][c] = *reinterpret_cast<lds_word*>((u[h][c] >> (30u - kWholeGuideBits)) & ~3u);
          }
        }
        const uint32_t base = (info[0] & 0xffffu) | info[1] << 16;
#pragma unroll
        for (uint32_t c = 0; c < CPL; ++c) {
          const uint32_t low = (d[0][c] + u[0][c]) >> (32u - kGuideBits), high = (d[1][c] + u[1][c]) >> (16u - kGuideBits);
          v[r * CPL + c] = ((high & 0xffff0000u) | low) + base;  // the upper 9 bits of either sum are its length
          own[c] += v[r * CPL + c];
          if (WHOLE) {
#pragma unroll
            for (uint32_t h = 0; h < 2; ++h) {
              const uint32_t l4 = ((w[h][c] + u[h][c]) >> (30u - kWholeGuideBits)) & ~3u;  // four times the length
              none[BINS == 2 ? 0 : h][c] += l4;
              atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(s_cnt) + l4), one[BINS == 2 ? 0 : h]);
            }
          }
        }
      }
#pragma unroll
      for (uint32_t c = 0; c < CPL; ++c) {
        note_halves(1, own[c], absent);
        if (WHOLE) {
#pragma unroll
          for (uint32_t h = 0; h < (BINS == 2 ? 1u : 2u); ++h) note(0, none[h][c] >> 2, absent);
        }
      }
      sort_columns<LG>(v, bit);
      uint32_t raster[C], snake[C / 2];
#pragma unroll
      for (uint32_t c = 0; c < C; ++c) {
        raster[c] = 0;
#pragma unroll
        for (uint32_t r = 0; r < RPL; ++r) raster[c] += v[r * C + c];
        raster[c] = (raster[c] ^ bit[0]) + uncomplement;
      }
#pragma unroll
      for (uint32_t c = 0; c < C / 2; ++c) {
        snake[c] = 0;
#pragma unroll
        for (uint32_t r = 0; r < RPL; ++r) snake[c] += (v[r * C + c] & ~odd[r]) | (v[r * C + C - 1u - c] & odd[r]);
        snake[c] = (snake[c] ^ bit[0]) + uncomplement;
      }
#pragma unroll
      for (uint32_t c = 0; c < C / 2; ++c) {  // the mirrored column of the snake has what is left of the two columns
        const uint32_t mirrored = raster[c] + raster[C - 1u - c] - snake[c];
        uint32_t x = raster[c] + from_partner<0>(raster[C - 1u - c]), y = snake[c] + from_partner<0>(mirrored);
#pragma unroll
        for (int b = 1; b < 6 - LG; ++b) x += partner_of(x, b), y += partner_of(y, b);
        note_halves(2, x, absent), note_halves(3, y, absent);
      }
    }
#pragma unroll
    for (int m = WHOLE ? 0 : 1; m < 4; ++m) {
      if (BINS == 1 && m > 0) {  // 0xffffffff: a wavefront that has seen no node
        lo[m] = lo[m] == 0xffffffffu ? lo[m] : min(lo[m] & 0xffffu, lo[m] >> 16);
        hi[m] = max(hi[m] & 0xffffu, hi[m] >> 16);
      }
      const uint32_t q = m == 0 ? LBS_NONE : m == 1 ? LBS_STRATIFIED : m == 2 ? LBS_LOCAL_RASTER : LBS_LOCAL_SNAKE;
      file_min_max(sh.fin, buf, q, lo[m], hi[m]);
    }
    if (WHOLE) {
      uint32_t glob_lo = 0xffffffffu, glob_hi = 0u;
      __syncthreads();
      whole_deal(P, s_cnt, s_gpu, &sh.base, sh.scan, glob_lo, glob_hi);
      file_min_max(sh.fin, buf, LBS_GLOBAL, glob_lo, glob_hi);
    }
    __syncthreads();  // also: this trial's last reads of s_cnt and s_gpu lie before the next trial's clearing
    finish_methods(P, sh.fin, sh.sum, buf, t, WHOLE, method, trial_min, trial_max);
  }
  if (tid < 2u * kMethods && (WHOLE || (tid >> 1) == method)) atomicAdd(&sums[WHOLE ? tid : (tid & 1u)], sh.sum[tid]);
}

// Which form a run of node-local methods takes: k_lbs_bins with one node at a time (the only one for nodes of 1, 2 and 16), with the columns in
// registers (nodes of 4 and 8: with two columns only 6 of the 21 stages would stay within a lane, 11 with four and 15 with eight, and
// sixteen are more columns than a group has lanes), or k_lbs_nodes with 8, 16 or 32 registers.
enum Form : uint32_t { kOneNode, kColumns, kNodes8, kNodes16, kNodes32, kForms };

// What it takes, in microseconds beyond what every launch does: workgroups start one every `launch` nanoseconds or, where that is more, one when the
// chip has got through a workgroup's trials; a wavefront's rounds in one trial, for the last workgroup; and, where the workgroups are more than
// fit on the chip at a time, what the last turn leaves idle.  A trial is a wavefront's rounds of `at_once` nodes (BINS == 1: pairs) at `each` (ns,
// whole chip), and a share of that for wavefronts without one in the last round, which weigh more where it is the only one.
//   Fitted to 4 180 runs, five methods at once and one alone, in every form: nodes of 4 and 8 in one and in two full bins, 2 to 256 nodes, 200
// to 100 000 trials (bins with padding and cells that have to be searched, nodes of 8 and five methods at once: 540 more).  The form
// taken is 0.3 and 0.4 % slower than the fastest of them on average (one method, all five).  Why the number of trials counts: 30 nodes of 4,
// batch 16, snake alone, us, columns / 16 registers: 1 700 trials 28.1 / 33.4 (eight workgroups a compute unit against six), 30 000
// 115.5 / 140.3, where so few nodes leave three wavefronts idle; 64 such nodes: 16 000 trials 111.2 / 124.8, 100 000 613 / 511.
struct Cost {
  uint32_t n;  // nodes, or pairs of nodes
  uint32_t gpn;
  bool two;    // bins
  uint32_t grid, n_cus;
  double trials;  // per workgroup
  bool whole, searched;
  double us(Form form) const {
    struct Entry {
      uint32_t at_once, resident;  // workgroups a compute unit
      double turn, trial, each;
    };
    static constexpr Entry one[] = {{1, 8, 0.58, 0.35, 0.2}, {8, 7, 1.7, 0.5, 1.3}, {8, 7, 1.3, 0.38, 1.11}, {16, 7, 2.0, 0.43, 1.77}, {32, 5, 3.2, 0.32, 3.31}};
    static constexpr Entry all[] = {{1, 6, 0.69, 1.2, 0.21}, {8, 5, 3.7, 1.56, 1.18}, {8, 6, 1.4, 1.8, 1.02}, {16, 6, 2.55, 1.55, 1.86}, {32, 5, 5.3, 2.37, 3.31}};
    Entry e = (whole ? all : one)[form];
    if (gpn == 4u) {
      if (form == kColumns) e = whole ? Entry{4, 6, 1.16, 1.02, 0.73} : Entry{4, 8, 0.75, 0.18, 0.74};
      if (form == kNodes16) e.resident = 6;
      if (form == kNodes32 && !whole && !two) e.resident = 6;
    } else if (whole && searched) {  // cells that have to be searched
      e = form == kOneNode ? Entry{1, 6, 0.89, 0.96, 0.32} : Entry{8, 5, 5.0, 1.6, 2.3};
    }
    const uint32_t rounds = (n + e.at_once - 1u) / e.at_once, turns = (rounds + kWaves - 1u) / kWaves, idle = turns * kWaves - rounds;
    const double trial = e.trial + e.each * (rounds + idle * (turns == 1u ? (whole ? 0.25 : 0.29) : (whole ? 0.21 : 0.05)));
    const uint32_t slots = e.resident * n_cus, last = grid > slots ? grid % slots : 0u;
    return e.turn * turns + 1e-3 * grid * std::max(whole ? 13.0 : 13.6, trial * trials) + (last != 0u ? (whole ? 2.15 : 1.2) * (slots - last) / slots : 0.0);
  }
};
Form pick_form(const Bins& B, const Params& P, uint32_t grid, uint32_t n_cus, bool whole, bool nodes) {
  const uint32_t gpn = P.gpus_per_node, n_nodes = P.n_gpus / gpn;
  if (gpn != 4u && gpn != 8u) return kOneNode;
  nodes = nodes && B.padded == 0 && P.flagged == 0;
  const Cost c{B.count == 2 ? n_nodes : (n_nodes + 1u) / 2u, gpn, B.count == 2, grid, n_cus, (double)P.n_trials / grid, whole, P.flagged != 0};
  Form best = kOneNode;
  double least = c.us(kOneNode);
  for (uint32_t f = kColumns; f < (nodes ? kForms : kNodes8); ++f) {
    if (f == kNodes8 && gpn == 4u) continue;  // that is the columns
    const double t = c.us((Form)f);
    if (t < least) least = t, best = (Form)f;
  }
  return best;
}

// k_lbs_bins for a run whose strata fit in L.count bins.
template <bool WHOLE>
auto bins_kernel(const Bins& L, const Params& P, Form form) {
  const bool two = L.count == 2;
  if (form == kColumns && P.gpus_per_node == 4) return two ? k_lbs_bins<2, 2, WHOLE> : k_lbs_bins<2, 1, WHOLE>;
  if (form == kColumns) return two ? k_lbs_bins<3, 2, WHOLE> : k_lbs_bins<3, 1, WHOLE>;
  return two ? k_lbs_bins<0, 2, WHOLE> : k_lbs_bins<0, 1, WHOLE>;
}

// Dynamic LDS of k_lbs_nodes, in bytes.
template <bool WHOLE>
size_t nodes_lds(const Params& P) {
  return sizeof(NodesShared<WHOLE>) + sizeof(uint32_t) * ((size_t)P.guide_words + (WHOLE ? kCountWords + P.n_gpus : 0u));
}

// k_lbs_nodes for a run that takes one of its forms; L: its rows.
template <bool WHOLE>
auto nodes_kernel(const Bins& B, const Params& P, Form form, Rows* L) {
  const uint32_t gpn = P.gpus_per_node, rows = 64u / gpn;
  *L = Rows{};
  for (uint32_t h = 0; h < B.count; ++h)
    for (uint32_t r = 0; r < rows; ++r) {
      const uint32_t j = B.slot[h][r];
      L->row[h][r] = P.slot_base[j] | (P.slot_guide[j] / kGuideSize) << 16 | j << 24;
      L->odd[h] |= (j & 1u) << r;
    }
  if (B.count == 2) {
    if (gpn == 4) return form == kNodes32 ? k_lbs_nodes<5, 2, 2, WHOLE> : k_lbs_nodes<4, 2, 2, WHOLE>;
    return form == kNodes32 ? k_lbs_nodes<5, 3, 2, WHOLE> : form == kNodes16 ? k_lbs_nodes<4, 3, 2, WHOLE> : k_lbs_nodes<3, 3, 2, WHOLE>;
  }
  if (gpn == 4) return form == kNodes32 ? k_lbs_nodes<5, 2, 1, WHOLE> : k_lbs_nodes<4, 2, 1, WHOLE>;
  return form == kNodes32 ? k_lbs_nodes<5, 3, 1, WHOLE> : form == kNodes16 ? k_lbs_nodes<4, 3, 1, WHOLE> : k_lbs_nodes<3, 3, 1, WHOLE>;
}

// Whether no LDS lies in front of the dynamic one in any k_lbs_nodes that takes the whole dataset's table for address 0.
hipError_t whole_tables_first(bool* first) {
  *first = true;
  for (const auto kernel : {k_lbs_nodes<4, 2, 1, true>, k_lbs_nodes<4, 2, 2, true>, k_lbs_nodes<5, 2, 1, true>, k_lbs_nodes<5, 2, 2, true>,
                            k_lbs_nodes<3, 3, 1, true>, k_lbs_nodes<3, 3, 2, true>, k_lbs_nodes<4, 3, 1, true>, k_lbs_nodes<4, 3, 2, true>,
                            k_lbs_nodes<5, 3, 1, true>, k_lbs_nodes<5, 3, 2, true>}) {
    hipFuncAttributes a;
    if (const hipError_t e = hipFuncGetAttributes(&a, reinterpret_cast<const void*>(kernel))) return e;
    if (a.sharedSizeBytes != 0) *first = false;
  }
  return hipSuccess;
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
  const auto first_over = [&](uint32_t index) {  // smallest length with more than `index` entries up to it
    while (cum[l] <= index) ++l;
    return l;
  };
  for (uint32_t ub = 0; ub < (1u << BITS); ++ub) {
    const uint64_t u_min = (uint64_t)ub << kLow, u_max = u_min + (1ull << kLow) - 1u;
    if (size == 0) {
      out[ub] = 0u;  // never drawn from
      continue;
    }
    const uint32_t l_min = first_over(before + (uint32_t)((u_min * size) >> 32));
    const uint32_t l_max = first_over(before + (uint32_t)((u_max * size) >> 32));
    if (l_max > l_min + 1u || l_max - base >= (1u << BITS) - 1u) {
      out[ub] = (kFlagged<BITS> | (l_min - 1u) | ((l_max - l_min) << 10)) - (uint32_t)u_min;
      flagged = true;
      continue;
    }
    out[ub] = ((l_min - base) << kLow) - (uint32_t)u_min;
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
    if (e == hipSuccess) e = whole_tables_first(&ds->whole_first);
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
    Rows rows;
    const Form form = local && L.count != 0 && !many_short ? pick_form(L, P, grid.x, ds->n_cus, false, true) : kOneNode;
    if (form >= kNodes8) {
      hipLaunchKernelGGL(nodes_kernel<false>(L, P, form, &rows), grid, block, nodes_lds<false>(P), s, P, rows, method, ds->d_guide, trial_min,
                         trial_max, ds_sums);
    } else if (local && L.count != 0 && !many_short) {
      hipLaunchKernelGGL(bins_kernel<false>(L, P, form), grid, block, sizeof(uint32_t) * tables, s, P, L, method, ds->d_cum, ds->d_guide, trial_min,
                         trial_max, ds_sums);
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
    Rows rows;
    const Form form = L.count != 0 ? pick_form(L, P, grid.x, ds->n_cus, true, ds->whole_first) : kOneNode;
    if (form >= kNodes8)
      hipLaunchKernelGGL(nodes_kernel<true>(L, P, form, &rows), grid, block, nodes_lds<true>(P), s, P, rows, 0u, ds->d_guide, trial_min, trial_max,
                         ds_sums);
    else if (L.count != 0)
      hipLaunchKernelGGL(bins_kernel<true>(L, P, form), grid, block, lds, s, P, L, 0u, ds->d_cum, ds->d_guide, trial_min, trial_max, ds_sums);
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
