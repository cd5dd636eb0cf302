// HIP kernels for gfx950 (MI355X): squared-norm partials, per-bucket finalize,
// in-place scale, the two launches of the per-bucket clip (with and without a plan),
// the (optionally clip-fused) Adam sweep, the whole fused step as one pipelined
// launch with its finish kernel, and LAMB's two sweeps.  Gradients are fp32, fp16 or bf16.
//
// All streaming kernels are table driven: the host cuts the bucket layout into
// chunks (<= chunk_elems consecutive elements of one tensor in one bucket,
// bca_internal.h) and workgroup w of a grid of G walks chunks c0+w, c0+w+G, ...
// Neighbouring workgroups therefore stream through neighbouring memory at the
// same time, and which workgroup handles a chunk never changes a result: a
// chunk's partial sums depend only on the chunk.  Two ways to fetch the table
// are compiled (STAGED): a persistent grid that copies its share of entries
// into LDS in slices, or uniform (scalar) loads of one entry per iteration,
// which is what a grid of one workgroup per chunk uses.
//
// Memory access: 128-bit loads/stores, lane-contiguous (a wavefront touches
// 1 KiB per instruction per array), several independent loads in flight per
// lane before first use, streaming (non-temporal) hints on data touched once.
// Arrays may start anywhere (gradients packed without padding next to aligned
// parameters are common): vectors are accessed at element alignment.  With
// gradients one element off their parameters' alignment the Adam sweep over 40 M
// elements takes 178 us (element by element, as it was before: 254; aligned: 187)
// and the fused step 196 us (243; 199).  No MFMA: nothing here is a contraction;
// the path is bound by HBM bandwidth.
//
// Arithmetic follows the paper's definitions: clipping-by-norm (Sec. 2.3)
// applied per bucket (Sec. 4.2, Alg. 1) and Adam (Alg. 1, last line; Kingma &
// Ba with bias correction, decoupled weight decay).  Every fp32 operation is
// written as an explicit multiply or fma so that the fused and the unfused
// paths produce the same bits.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "bca_internal.h"

namespace bca {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// ---- streaming accesses ---------------------------------------------------------
// NT = non-temporal: data that is touched once per launch is loaded and stored
// with the streaming hint, which raises HBM throughput on gfx950 and keeps such
// lines from displacing reusable ones in L2 / Infinity Cache.
//
// Tensor addresses come out of the chunk table as integers, so the compiler cannot tell that they are global
// memory and would emit flat accesses; those may complete out of order, which forces a full wait
// (vmcnt(0) lgkmcnt(0)) before the first use of any of them and leaves only two or three of a batch of
// loads in flight.  Every access to tensor memory therefore goes through a pointer that is explicitly in the
// global address space: global_load / global_store, counted waits, all loads of a batch in flight.
// loads_issued(): nothing is scheduled across this point, so a batch of loads written before it is issued as a
// whole before the first instruction that uses one of them (left to itself the scheduler interleaves loads and
// uses in pairs, which leaves two loads in flight where eight or sixteen were meant).
__device__ __forceinline__ void loads_issued() { __builtin_amdgcn_sched_barrier(0); }
#define BCA_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ BCA_GLOBAL T* as_global(T* p) {
  return (BCA_GLOBAL T*)p;
}
// A vector is accessed wherever its first element lies: gfx950 runs in unaligned access mode, so a 128-bit (64-bit)
// access needs no more than its element's alignment, and telling the compiler so is all it takes to get the same
// global_load_dwordx4 / dwordx2 as for aligned data.  A wavefront's access then touches one cache line more.
template <typename T>
struct Anywhere;
template <>
struct Anywhere<f32x4> {
  typedef f32x4 type __attribute__((aligned(4)));
};
template <>
struct Anywhere<f16x4> {
  typedef f16x4 type __attribute__((aligned(2)));
};
template <>
struct Anywhere<f16x8> {
  typedef f16x8 type __attribute__((aligned(2)));
};
template <>
struct Anywhere<u16x4> {
  typedef u16x4 type __attribute__((aligned(2)));
};
template <>
struct Anywhere<u16x8> {
  typedef u16x8 type __attribute__((aligned(2)));
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <>
struct Anywhere<u32x4> {
  typedef u32x4 type __attribute__((aligned(4)));
};
template <bool NT, typename T>
__device__ __forceinline__ T ldv(const T* p) {
  typedef typename Anywhere<T>::type U;
  if constexpr (NT) return __builtin_nontemporal_load((const BCA_GLOBAL U*)p);
  else return *(const BCA_GLOBAL U*)p;
}
template <bool NT, typename T>
__device__ __forceinline__ void stv(T* p, T x) {
  typedef typename Anywhere<T>::type U;
  if constexpr (NT) __builtin_nontemporal_store(x, (BCA_GLOBAL U*)p);
  else *(BCA_GLOBAL U*)p = x;
}

// Pieces of eight 16-bit elements that start in the middle of a 32-bit word: p (piece 0 of this lane), p + stride, ...; lane
// l + 1 has the pieces behind those of lane l.  128-bit loads that start on words of 32 bits cost what aligned ones do; from the middle of
// one they are 10 to 20 % slower (squared norms of 128 M bf16 one element off 45.5 us before any of this, with loads from
// where the pieces start 53.7, like this 45.1; out of the caches 53.0 / 59.4 / 48.3; clip of 16 M 16.9 / 19.9 / 17.1).  So a lane loads
// the words from the one that holds its first element on, takes the word behind them from the next lane (lane 63 loads it), and
// shifts them into place.  Every word that is read holds an element of the piece.
template <bool NT, uint32_t U, typename W>
__device__ __forceinline__ void ld_odd(W (&x)[U], const W* p, uint32_t stride) {
  const uint64_t a = reinterpret_cast<uint64_t>(p) - 2u;
  u32x4 w[U];
  uint32_t next[U] = {};
#pragma unroll
  for (uint32_t u = 0; u < U; ++u) w[u] = ldv<NT>(reinterpret_cast<const u32x4*>(a) + u * stride);
  if ((threadIdx.x & 63u) == 63u) {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const BCA_GLOBAL uint32_t* q = (const BCA_GLOBAL uint32_t*)(a + 16u) + u * stride * 4u;
      if constexpr (NT) next[u] = __builtin_nontemporal_load(q);
      else next[u] = *q;
    }
  }
  loads_issued();
#pragma unroll
  for (uint32_t u = 0; u < U; ++u) {
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)next[u], (int)w[u].x, 0x130, 0xf, 0xf, false);  // wave_shl:1
    u32x4 r;
    r.x = __builtin_amdgcn_alignbit(w[u].y, w[u].x, 16u), r.y = __builtin_amdgcn_alignbit(w[u].z, w[u].y, 16u);
    r.z = __builtin_amdgcn_alignbit(w[u].w, w[u].z, 16u), r.w = __builtin_amdgcn_alignbit(y, w[u].w, 16u);
    x[u] = __builtin_bit_cast(W, r);
  }
}

// ---- chunk table access -----------------------------------------------------------

struct Entry {  // one chunk, in registers (uniform across the workgroup)
  uint64_t g, p, m, v;
  uint32_t len, bucket, tensor, flags;
};

__device__ __forceinline__ Entry read_entry(const Chunk* e) {
  Entry r;
  r.g = e->g, r.p = e->p, r.m = e->m, r.v = e->v, r.len = e->len, r.bucket = e->bucket;
  r.tensor = e->tensor, r.flags = e->flags;
  return r;
}

// Number of chunks workgroup w of G owns out of n under interleaved assignment.
__device__ __forceinline__ uint32_t my_chunk_count(uint32_t n, uint32_t w, uint32_t G) {
  return n > w ? (n - w + G - 1) / G : 0u;
}

// Copy entries  table[c0 + w + (first + e) * G], e in [0, cnt)  into LDS.
__device__ __forceinline__ void stage_slice(Chunk* s_tab, const Chunk* table, uint32_t c0, uint32_t w, uint32_t G,
                                            uint32_t first, uint32_t cnt) {
  const uint4* src = reinterpret_cast<const uint4*>(table);
  uint4* dst = reinterpret_cast<uint4*>(s_tab);
  for (uint32_t q = threadIdx.x; q < cnt * 3u; q += kBlock) {
    const uint32_t e = q / 3u, piece = q - e * 3u;
    const uint64_t ci = (uint64_t)c0 + w + (uint64_t)(first + e) * G;
    dst[q] = src[ci * 3u + piece];
  }
}

// Calls body(entry, chunk_index) for every chunk of this workgroup.
template <bool STAGED, typename F>
__device__ __forceinline__ void for_each_chunk(const Chunk* __restrict__ table, uint32_t c0, uint32_t n, F body) {
  const uint32_t w = blockIdx.x, Gn = gridDim.x;
  if constexpr (STAGED) {
    __shared__ Chunk s_tab[kSlice];
    const uint32_t mine = my_chunk_count(n, w, Gn);
    for (uint32_t first = 0; first < mine; first += kSlice) {
      const uint32_t cnt = min(kSlice, mine - first);
      stage_slice(s_tab, table, c0, w, Gn, first, cnt);
      __syncthreads();
      for (uint32_t e = 0; e < cnt; ++e) body(read_entry(&s_tab[e]), c0 + w + (first + e) * Gn);
      __syncthreads();
    }
  } else {
    for (uint32_t i = w; i < n; i += Gn) body(read_entry(&table[c0 + i]), c0 + i);
  }
}

// ---- gradient access by storage type -----------------------------------------

template <int GDT>
struct Grad;

// `wide` is the 128-bit piece the squared-norm pass loads; widen() turns it into
// its VE fp32 values (exactly).
template <>
struct Grad<BCA_GRAD_F32> {
  typedef float elem;
  typedef f32x4 wide;
  static constexpr uint32_t VE = 4;
  static __device__ __forceinline__ void widen(const wide& x, float (&f)[VE]) {
    f[0] = x.x, f[1] = x.y, f[2] = x.z, f[3] = x.w;
  }
  static __device__ __forceinline__ wide narrow(const float (&f)[VE]) {
    wide x;
    x.x = f[0], x.y = f[1], x.z = f[2], x.w = f[3];
    return x;
  }
  template <bool NT>
  static __device__ __forceinline__ f32x4 load4(const void* base, uint32_t vec) {
    return ldv<NT>(reinterpret_cast<const f32x4*>(base) + vec);
  }
  template <bool NT>
  static __device__ __forceinline__ void store4(void* base, uint32_t vec, f32x4 x) {
    stv<NT>(reinterpret_cast<f32x4*>(base) + vec, x);
  }
  static __device__ __forceinline__ float load1(const void* base, uint32_t i) {
    return as_global(reinterpret_cast<const float*>(base))[i];
  }
  static __device__ __forceinline__ void store1(void* base, uint32_t i, float x) {
    as_global(reinterpret_cast<float*>(base))[i] = x;
  }
};

template <>
struct Grad<BCA_GRAD_F16> {
  typedef _Float16 elem;
  typedef f16x8 wide;
  static constexpr uint32_t VE = 8;
  static __device__ __forceinline__ void widen(const wide& x, float (&f)[VE]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = (float)x[q];
  }
  // fp16 -> fp32 is exact (subnormals included); fp32 -> fp16 rounds to nearest even.  What is stored is the
  // fp32 value rounded once more: settled() keeps the compiler from folding the multiplication that made the
  // value into the conversion (a mixed-precision multiply rounds the exact product to fp16 in one step, which
  // differs from the two roundings on ties of the fp32 product, about one stored value in a thousand).
  static __device__ __forceinline__ float settled(float x) {
    asm volatile("" : "+v"(x));
    return x;
  }
  static __device__ __forceinline__ wide narrow(const float (&f)[VE]) {  // the rounding of store4 / store1
    wide x;
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = (_Float16)settled(f[q]);
    return x;
  }
  template <bool NT>
  static __device__ __forceinline__ f32x4 load4(const void* base, uint32_t vec) {
    const f16x4 h = ldv<NT>(reinterpret_cast<const f16x4*>(base) + vec);
    f32x4 r;
    r.x = (float)h.x, r.y = (float)h.y, r.z = (float)h.z, r.w = (float)h.w;
    return r;
  }
  template <bool NT>
  static __device__ __forceinline__ void store4(void* base, uint32_t vec, f32x4 x) {
    f16x4 h;
    h.x = (_Float16)settled(x.x), h.y = (_Float16)settled(x.y), h.z = (_Float16)settled(x.z), h.w = (_Float16)settled(x.w);
    stv<NT>(reinterpret_cast<f16x4*>(base) + vec, h);
  }
  static __device__ __forceinline__ float load1(const void* base, uint32_t i) {
    return (float)as_global(reinterpret_cast<const _Float16*>(base))[i];
  }
  static __device__ __forceinline__ void store1(void* base, uint32_t i, float x) {
    as_global(reinterpret_cast<_Float16*>(base))[i] = (_Float16)settled(x);
  }
};

// bfloat16 is the upper half of a binary32: widening appends 16 zero bits (exact);
// narrowing rounds to nearest, ties to even, in integer arithmetic (the carry out of
// the fraction moves to the exponent and ends at infinity, as it should); NaN stays
// NaN with the quiet bit set.
__device__ __forceinline__ float bf16_to_f32(unsigned short h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ unsigned short f32_to_bf16(float x) {
  const uint32_t u = __float_as_uint(x);
  if (x != x) return (unsigned short)((u >> 16) | 0x40u);
  return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

template <>
struct Grad<BCA_GRAD_BF16> {
  typedef unsigned short elem;
  typedef u16x8 wide;
  static constexpr uint32_t VE = 8;
  static __device__ __forceinline__ void widen(const wide& x, float (&f)[VE]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = bf16_to_f32(x[q]);
  }
  static __device__ __forceinline__ wide narrow(const float (&f)[VE]) {
    wide x;
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = f32_to_bf16(f[q]);
    return x;
  }
  template <bool NT>
  static __device__ __forceinline__ f32x4 load4(const void* base, uint32_t vec) {
    const u16x4 h = ldv<NT>(reinterpret_cast<const u16x4*>(base) + vec);
    f32x4 r;
    r.x = bf16_to_f32(h.x), r.y = bf16_to_f32(h.y), r.z = bf16_to_f32(h.z), r.w = bf16_to_f32(h.w);
    return r;
  }
  template <bool NT>
  static __device__ __forceinline__ void store4(void* base, uint32_t vec, f32x4 x) {
    u16x4 h;
    h.x = f32_to_bf16(x.x), h.y = f32_to_bf16(x.y), h.z = f32_to_bf16(x.z), h.w = f32_to_bf16(x.w);
    stv<NT>(reinterpret_cast<u16x4*>(base) + vec, h);
  }
  static __device__ __forceinline__ float load1(const void* base, uint32_t i) {
    return bf16_to_f32(as_global(reinterpret_cast<const unsigned short*>(base))[i]);
  }
  static __device__ __forceinline__ void store1(void* base, uint32_t i, float x) {
    as_global(reinterpret_cast<unsigned short*>(base))[i] = f32_to_bf16(x);
  }
};

// LAMB's sweeps: elements to handle one by one so that the vectors that follow are 16-byte aligned in p, m and v
// alike, where such a head exists (0 .. 3 elements).  Their cacheable moment stores suffer from lines written in two
// parts: 40 M elements with all arrays one element off a 16-byte boundary take 275 us with the head and 290 without.
// The Adam sweeps, whose stores stream, are better off without one (190 against 200 us on the same arrays).
__device__ __forceinline__ uint32_t vector_head(uint32_t len, uint64_t p, uint64_t m, uint64_t v) {
  if (((p ^ m) | (p ^ v)) & 15u) return 0;
  const uint32_t h = (uint32_t)((16u - (p & 15u)) & 15u) / 4u;
  return h < len ? h : len;
}

// ---- wavefront reduction (fixed order) ----------------------------------------

// Sums by butterfly, distances 32, 16, 8, 4, 2, 1.  Lanes meet by permlane swaps (32, 16) and by DPP rotations inside rows of 16:
// with the value 8 lanes on already added, rotating by 4 brings the one 4 lanes across, and so on down.  Every one of these launches
// ends in a chain of such sums, and a move is a vector instruction where a shuffle is a trip through LDS: fused steps of 17 K and 0.5 M
// elements, one plan called again and again, 7.2 -> 6.8 and 8.6 -> 8.2 us (five turns; where inputs change from pass to pass no difference:
// 5.95 -> 5.94), LAMB on 335 M elements (two sums a chunk) 1 862 -> 1 850.
__device__ __forceinline__ double join(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo); }
// Rows 2, 3 of a and rows 0, 1 of b change places, then the two are added: lanes 0 .. 31 hold the sums of a's lanes 32 apart, lanes
// 32 .. 63 those of b's.  add16: the same with the odd rows of a, the even rows of b and lanes 16 apart.
__device__ __forceinline__ double add32(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return join(lo[0], hi[0]) + join(lo[1], hi[1]);
}
__device__ __forceinline__ double add16(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return join(lo[0], hi[0]) + join(lo[1], hi[1]);
}
template <int CTRL>
__device__ __forceinline__ double add_rotated(double a) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, CTRL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, false);
  return a + join(lo, hi);
}
__device__ __forceinline__ double row_sum(double x) {
  return add_rotated<0x121>(add_rotated<0x122>(add_rotated<0x124>(add_rotated<0x128>(x))));  // row_ror by 8, 4, 2, 1
}
__device__ __forceinline__ double wave_sum(double x) {
  x = add32(x, x);
  return row_sum(add16(x, x));
}

// ---- squared-norm partials ------------------------------------------------------

// Adds the squares of one 128-bit piece to the lane's four fp32 accumulators: element q of the piece goes to
// accumulator q mod 4, in element order.  Every squared-norm path goes through this one function, so that a
// chunk's partial sums do not depend on which kernel computed them.
template <int GDT>
__device__ __forceinline__ void add_squares(const typename Grad<GDT>::wide& x, float& a0, float& a1, float& a2, float& a3) {
  constexpr uint32_t VE = Grad<GDT>::VE;
  float f[VE];
  Grad<GDT>::widen(x, f);
#pragma unroll
  for (uint32_t q = 0; q < VE; q += 4) {
    a0 = __fmaf_rn(f[q], f[q], a0), a1 = __fmaf_rn(f[q + 1], f[q + 1], a1);
    a2 = __fmaf_rn(f[q + 2], f[q + 2], a2), a3 = __fmaf_rn(f[q + 3], f[q + 3], a3);
  }
}

// Sum of g^2 over the part of a chunk this wavefront reads, in fp64 (same value
// in every lane).  Per lane the squares are accumulated in fp32 (four independent
// accumulators, at most chunk_elems/1024 terms each), then the lanes are combined
// in fp64 by butterfly shuffles.  Wavefronts never wait for each other.
// LOADS: 128-bit loads in flight per lane, ODD: whether 16-bit elements off 32-bit words go by ld_odd (the result depends on
// neither).
template <int GDT, bool NT, uint32_t LOADS = 8, bool ODD = true>
__device__ __forceinline__ double sqnorm_chunk(const Entry& en) {
  typedef Grad<GDT> G;
  constexpr uint32_t VE = G::VE;  // elements per 128-bit load: 4 (fp32) or 8 (fp16, bf16)
  constexpr uint32_t whole = kDefaultChunkNorm / (VE * kBlock), U = LOADS < whole ? LOADS : whole;  // no more than a chunk has
  const uint32_t tid = threadIdx.x;
  const uint64_t ga = en.g;
  const uint32_t len = en.len;
  const uint32_t nvec = len / VE;
  const uint32_t tail0 = nvec * VE;
  const void* gbase = reinterpret_cast<const void*>(ga);
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;

  typedef typename G::wide wide;
  const wide* gw = reinterpret_cast<const wide*>(ga);
  // Lane t adds pieces t, t + 256, t + 512, ... in that order.  They are fetched U at a time; a slot past the end
  // of the chunk holds zeros, whose squares leave the (non-negative) accumulators as they are.
  for (uint32_t base = 0; base < nvec; base += kBlock * U) {
    const uint32_t j0 = base + tid;
    wide x[U];
    if (base + kBlock * U <= nvec) {
      bool odd = false;
      if constexpr (ODD && VE == 8) {
        odd = (ga & 2u) != 0;
        if (odd) ld_odd<NT>(x, gw + j0, kBlock);
      }
      if (!odd) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) x[u] = ldv<NT>(gw + j0 + u * kBlock);
      }
    } else {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t j = j0 + u * kBlock;
        x[u] = wide{};
        if (j < nvec) x[u] = ldv<NT>(gw + j);
      }
    }
    loads_issued();
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) add_squares<GDT>(x[u], a0, a1, a2, a3);
  }
  // the last, fewer than VE, elements one by one
  for (uint32_t i = tail0 + tid; i < len; i += kBlock) {
    const float x = G::load1(gbase, i);
    a1 = __fmaf_rn(x, x, a1);
  }
  const double lane = ((double)a0 + (double)a1) + ((double)a2 + (double)a3);
  return wave_sum(lane);
}

// kWaves partials (fp64) per chunk, one per wavefront.  The finalize pass adds a
// bucket's partials in a fixed order.
template <int GDT, bool NT, bool STAGED, uint32_t U>
__global__ __launch_bounds__(kBlock) void k_sqnorm(const Chunk* __restrict__ table, uint32_t c0, uint32_t n,
                                                    double* __restrict__ partials, int32_t* status) {
  const uint32_t tid = threadIdx.x;
  if (status != nullptr && blockIdx.x == 0 && tid == 0) *status = 0;  // finalize ORs into it later on this stream
  for_each_chunk<STAGED>(table, c0, n, [&](const Entry& en, uint32_t ci) {
    const double ws = sqnorm_chunk<GDT, NT, U>(en);
    if ((tid & 63u) == 0) partials[(uint64_t)ci * kWaves + (tid >> 6)] = ws;
  });
}

// ---- clip coefficient -----------------------------------------------------------

// Sec. 2.3: if ||g|| >= c the gradient is multiplied by c / ||g||, else left
// alone.  The quotient is taken in fp64 from the fp32 norm and rounded once.
// A threshold that is not a positive number means "no clipping" and is flagged.
__device__ __forceinline__ float clip_coef(float norm, float c, int32_t& status) {
  if (!(fabsf(norm) <= 3.402823466e38f)) status |= BCA_STATUS_NONFINITE;  // Inf or NaN
  if (!(c > 0.f)) {
    status |= BCA_STATUS_BAD_THRESHOLD;
    return 1.f;
  }
  if (norm >= c) return (float)((double)c / (double)norm);
  return 1.f;
}

// The sum of partials[lo .. hi) in THE order every path uses (thread t adds lo + t, lo + t + 256, ... one after the
// other, lanes by butterfly, wavefronts in index order), computed by the whole workgroup; loads are issued eight
// at a time before the first addition, a slot past the end adding +0.0.  Valid in thread 0.
__device__ __forceinline__ double sum_partials(const double* __restrict__ partials, uint64_t lo, uint64_t hi, double* s_w) {
  const uint32_t tid = threadIdx.x;
  double s = 0.0;
  for (uint64_t i = lo + tid; i < hi; i += 8u * kBlock) {
    double part[8];
#pragma unroll
    for (uint32_t q = 0; q < 8u; ++q) {
      const uint64_t j = i + (uint64_t)q * kBlock;
      part[q] = j < hi ? partials[j] : 0.0;
    }
#pragma unroll
    for (uint32_t q = 0; q < 8u; ++q) s += part[q];
  }
  s = wave_sum(s);
  if ((tid & 63u) == 0) s_w[tid >> 6] = s;
  __syncthreads();
  return ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
}

// One workgroup per bucket: threads take the bucket's partials in strides of 256
// in fp64, lanes are combined by a butterfly, the four wavefronts through LDS in
// index order.  Same order on every run, so norms are reproducible.
__global__ __launch_bounds__(kBlock) void k_finalize(const double* __restrict__ partials,
                                                      const uint32_t* __restrict__ bucket_chunk_off, uint32_t b0,
                                                      const float* __restrict__ thresholds, float* __restrict__ norms,
                                                      float* __restrict__ coefs, int32_t* status,
                                                      double* __restrict__ bucket_sq) {
  __shared__ double s_w[kWaves];
  const uint32_t b = b0 + blockIdx.x;
  const uint64_t lo = (uint64_t)bucket_chunk_off[b] * kWaves, hi = (uint64_t)bucket_chunk_off[b + 1] * kWaves;
  const double tot = sum_partials(partials, lo, hi, s_w);
  if (threadIdx.x == 0) {
    const float norm = (float)sqrt(tot);
    norms[b] = norm;
    if (bucket_sq != nullptr) bucket_sq[b] = tot;
    if (thresholds != nullptr) {
      int32_t st = 0;
      const float coef = clip_coef(norm, thresholds[b], st);
      coefs[b] = coef;
      if (st != 0 && status != nullptr) atomicOr(status, st);
    }
  }
}

// Whole-gradient clipping (Sec. 3.2's baselines): the buckets' sums of squares
// are added in index order in fp64, the clipping rule of Sec. 2.3 is applied
// once with the single threshold *c, and every bucket gets that coefficient.
// One workgroup; ORs its status bits into *status.
__global__ __launch_bounds__(kBlock) void k_whole_coef(const double* __restrict__ bucket_sq, uint32_t n_buckets,
                                                        const float* __restrict__ c, float* __restrict__ whole_norm,
                                                        float* __restrict__ coefs, int32_t* status) {
  __shared__ double s_w[kWaves];
  __shared__ float s_coef;
  double s = 0.0;
  for (uint32_t b = threadIdx.x; b < n_buckets; b += kBlock) s += bucket_sq[b];
  s = wave_sum(s);
  if ((threadIdx.x & 63u) == 0) s_w[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float norm = (float)sqrt(((s_w[0] + s_w[1]) + s_w[2]) + s_w[3]);
    int32_t st = 0;
    s_coef = clip_coef(norm, *c, st);
    *whole_norm = norm;
    if (st != 0) atomicOr(status, st);
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < n_buckets; b += kBlock) coefs[b] = s_coef;
}

// Coefficients from norms the caller supplies (unfused path).  One workgroup;
// writes (not ORs) the status word of this call.
__global__ __launch_bounds__(kBlock) void k_coefs(uint32_t b0, uint32_t b1, const float* __restrict__ thresholds,
                                                   const float* __restrict__ norms, float* __restrict__ coefs,
                                                   int32_t* status) {
  __shared__ int32_t s_st;
  if (threadIdx.x == 0) s_st = 0;
  __syncthreads();
  int32_t st = 0;
  for (uint32_t b = b0 + threadIdx.x; b < b1; b += kBlock) coefs[b] = clip_coef(norms[b], thresholds[b], st);
  if (st != 0) atomicOr(&s_st, st);
  __syncthreads();
  if (threadIdx.x == 0 && status != nullptr) *status = s_st;
}

// ---- in-place scale -------------------------------------------------------------

// g <- coef * g over one chunk, in the gradient's storage type (Alg. 1, the
// assignment under the if).
template <int GDT, uint32_t U, bool NT>
__device__ __forceinline__ void scale_chunk(const Entry& en, float coef) {
  typedef Grad<GDT> G;
  const uint32_t tid = threadIdx.x;
  const uint32_t len = en.len;
  const uint32_t nvec = len / 4u;
  const uint32_t tail0 = nvec * 4u;
  void* gv = reinterpret_cast<void*>(en.g);
  for (uint32_t base = 0; base < nvec; base += kBlock * U) {
    const uint32_t j0 = base + tid;
    if (base + kBlock * U <= nvec) {
      f32x4 x[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) x[u] = G::template load4<NT>(gv, j0 + u * kBlock);
      loads_issued();
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) G::template store4<NT>(gv, j0 + u * kBlock, x[u] * coef);
    } else {
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t j = j0 + u * kBlock;
        if (j < nvec) G::template store4<NT>(gv, j, G::template load4<NT>(gv, j) * coef);
      }
    }
  }
  for (uint32_t i = tail0 + tid; i < len; i += kBlock) G::store1(gv, i, G::load1(gv, i) * coef);
}

// Buckets with coef_b == 1 are not read at all.
template <int GDT, uint32_t U, bool NT, bool STAGED>
__global__ __launch_bounds__(kBlock) void k_scale(const Chunk* __restrict__ table, uint32_t c0, uint32_t n,
                                                   const float* __restrict__ coefs) {
  for_each_chunk<STAGED>(table, c0, n, [&](const Entry& en, uint32_t) {
    const float coef = coefs[en.bucket];
    if (coef != 1.f) scale_chunk<GDT, U, NT>(en, coef);
  });
}

// ---- Adam -----------------------------------------------------------------------

// One element of  theta <- ADAM(theta, eta, G)  (Alg. 1, last line):
//   m <- b1 m + (1-b1) g;  v <- b2 v + (1-b2) g^2
//   p <- p - lr * ( mhat / (sqrt(vhat) + eps) + wd p ),  mhat = m/(1-b1^t), vhat = v/(1-b2^t)
// Division and square root are the correctly rounded ones.
// wd is the weight decay that applies to the element's tensor: k.wd, or 0 for a
// tensor the decay mask exempts.
// The constants a kernel works with: those passed by value, or the device copy they point to.
__device__ __forceinline__ AdamK resolve(const AdamK& a) {
  if (a.from != nullptr) return *a.from;
  return a;
}

// Hyper-parameters in device memory -> the sweeps' constants, as the host derives them from a bca_adam.  The call's other launches
// wait for this one, whose time is that of a power in fp64: lane 0 takes beta1's while lane 1 takes beta2's.
__global__ __launch_bounds__(64) void k_hyper(const bca_adam_device* __restrict__ dev, AdamK* __restrict__ out) {
  if (threadIdx.x > 1) return;
  const double t = (double)dev->step;
  const float rbc = (float)(1.0 / (1.0 - pow(threadIdx.x == 0 ? dev->beta1 : dev->beta2, t)));
  const float rbc2 = __shfl(rbc, 1, 64);
  if (threadIdx.x != 0) return;
  AdamK k;
  k.b1 = (float)dev->beta1, k.omb1 = (float)(1.0 - dev->beta1);
  k.b2 = (float)dev->beta2, k.omb2 = (float)(1.0 - dev->beta2);
  k.rbc1 = rbc, k.rbc2 = rbc2;
  k.eps = (float)dev->eps;
  k.neg_lr = (float)(-dev->lr);
  k.wd = (float)dev->weight_decay;
  k.lr = dev->lr;
  k.from = nullptr;
  *out = k;
}

__device__ __forceinline__ void adam_moments(float g, float& m, float& v, const AdamK& k) {
  m = __fmaf_rn(k.b1, m, k.omb1 * g);
  v = __fmaf_rn(k.b2, v, k.omb2 * (g * g));
}
// mhat / (sqrt(vhat) + eps) + wd p: the bracket of Adam's parameter update, which is
// also LAMB's update direction.
__device__ __forceinline__ float adam_direction(float p, float m, float v, const AdamK& k, float wd) {
  const float mhat = m * k.rbc1;
  const float vhat = v * k.rbc2;
  const float denom = __fsqrt_rn(vhat) + k.eps;
  return __fmaf_rn(wd, p, __fdiv_rn(mhat, denom));
}
__device__ __forceinline__ void adam1(float g, float& p, float& m, float& v, const AdamK& k, float wd) {
  adam_moments(g, m, v, k);
  p = __fmaf_rn(k.neg_lr, adam_direction(p, m, v, k, wd), p);
}

__device__ __forceinline__ void adam4(f32x4 g, f32x4& p, f32x4& m, f32x4& v, const AdamK& k, float wd) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float pi = p[i], mi = m[i], vi = v[i];
    adam1(g[i], pi, mi, vi, k, wd);
    p[i] = pi, m[i] = mi, v[i] = vi;
  }
}

__device__ __forceinline__ float chunk_wd(const Entry& en, const AdamK& k) {
  return (en.flags & kChunkNoDecay) ? 0.f : k.wd;
}

// The read-modify-write sweep over one chunk.  coef != 1 only on the fused path:
// ghat = coef_b * g is formed in registers (one fp32 multiply, so it equals what
// k_scale would have stored for fp32 gradients); WB: ghat, rounded to the gradient
// type, also replaces g.  p, m, v are touched once per sweep and always stream;
// GNT says whether g streams too.
template <int GDT, bool FUSED, bool WB, uint32_t U, bool GNT>
__device__ __forceinline__ void adam_chunk(const Entry& en, float coef, const AdamK& k) {
  typedef Grad<GDT> G;
  constexpr bool NT = true;
  const uint32_t tid = threadIdx.x;
  const uint64_t ga = en.g, pa = en.p, ma = en.m, va = en.v;
  const uint32_t len = en.len;
  const bool wb = WB && coef != 1.f;
  const float wd = chunk_wd(en, k);
  const uint32_t nvec = len / 4u;
  const uint32_t tail0 = nvec * 4u;
  void* gv = reinterpret_cast<void*>(ga);
  f32x4* pv = reinterpret_cast<f32x4*>(pa);
  f32x4* mv = reinterpret_cast<f32x4*>(ma);
  f32x4* vv = reinterpret_cast<f32x4*>(va);

  for (uint32_t base = 0; base < nvec; base += kBlock * U) {
    const uint32_t j0 = base + tid;
    if (base + kBlock * U <= nvec) {
      f32x4 g[U], p[U], m[U], v[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) g[u] = G::template load4<GNT>(gv, j0 + u * kBlock);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) p[u] = ldv<NT>(pv + j0 + u * kBlock);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) m[u] = ldv<NT>(mv + j0 + u * kBlock);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) v[u] = ldv<NT>(vv + j0 + u * kBlock);
      loads_issued();
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        if constexpr (FUSED) g[u] = g[u] * coef;
        adam4(g[u], p[u], m[u], v[u], k, wd);
        const uint32_t j = j0 + u * kBlock;
        stv<NT>(pv + j, p[u]), stv<NT>(mv + j, m[u]), stv<NT>(vv + j, v[u]);
        if (wb) G::template store4<GNT>(gv, j, g[u]);
      }
    } else {
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t j = j0 + u * kBlock;
        if (j < nvec) {
          f32x4 g = G::template load4<GNT>(gv, j), p = ldv<NT>(pv + j), m = ldv<NT>(mv + j), v = ldv<NT>(vv + j);
          if constexpr (FUSED) g = g * coef;
          adam4(g, p, m, v, k, wd);
          stv<NT>(pv + j, p), stv<NT>(mv + j, m), stv<NT>(vv + j, v);
          if (wb) G::template store4<GNT>(gv, j, g);
        }
      }
    }
  }
  // the last, fewer than four, elements
  BCA_GLOBAL float* p1 = as_global(reinterpret_cast<float*>(pa));
  BCA_GLOBAL float* m1 = as_global(reinterpret_cast<float*>(ma));
  BCA_GLOBAL float* v1 = as_global(reinterpret_cast<float*>(va));
  for (uint32_t i = tail0 + tid; i < len; i += kBlock) {
    float g = G::load1(gv, i), p = p1[i], m = m1[i], v = v1[i];
    if constexpr (FUSED) g = g * coef;
    adam1(g, p, m, v, k, wd);
    p1[i] = p, m1[i] = m, v1[i] = v;
    if (wb) G::store1(gv, i, g);
  }
}

// One full chunk (four elements a thread) of the fused sweep whose coefficient is not known yet: everything is loaded first, then
// wait() says whether there is a coefficient, and leaves it in *coef.  The arithmetic is adam_chunk's.
template <int GDT, bool WB, typename W>
__device__ __forceinline__ void adam_chunk_early(const Entry& en, const AdamK& k, const float* coef, W wait) {
  typedef Grad<GDT> G;
  const uint32_t tid = threadIdx.x;
  f32x4* pv = reinterpret_cast<f32x4*>(en.p) + tid;
  f32x4* mv = reinterpret_cast<f32x4*>(en.m) + tid;
  f32x4* vv = reinterpret_cast<f32x4*>(en.v) + tid;
  void* gv = reinterpret_cast<void*>(en.g);
  f32x4 g = G::template load4<false>(gv, tid), p = ldv<true>(pv), m = ldv<true>(mv), v = ldv<true>(vv);
  loads_issued();
  if (!wait()) return;
  const float c = *coef;
  g = g * c;
  adam4(g, p, m, v, k, chunk_wd(en, k));
  stv<true>(pv, p), stv<true>(mv, m), stv<true>(vv, v);
  if (WB && c != 1.f) G::template store4<false>(gv, tid, g);
}

// The chunk that comes i-th (AdamOrder).
__device__ __forceinline__ uint32_t adam_chunk_of(uint32_t i, uint32_t n, AdamOrder order) {
  if (order == AdamOrder::kTable) return i;
  const uint32_t at = i % (8u * kXcdRun), base = i - at;
  if (n - base >= 8u * kXcdRun) return base + (at % 8u) * kXcdRun + at / 8u;
  return i;
}

template <int GDT, bool FUSED, bool WB, uint32_t U, bool GNT, bool STAGED>
__global__ __launch_bounds__(kBlock) void k_adam(const Chunk* __restrict__ table, uint32_t c0, uint32_t n,
                                                  const float* __restrict__ coefs, const int32_t* skip_status,
                                                  const AdamK ka, AdamOrder order) {
  if (skip_status != nullptr && (*skip_status & BCA_STATUS_NONFINITE)) return;
  const AdamK k = resolve(ka);
  const auto sweep = [&](const Entry& en, uint32_t) {
    float coef = 1.f;
    if constexpr (FUSED) coef = coefs[en.bucket];
    adam_chunk<GDT, FUSED, WB, U, GNT>(en, coef, k);
  };
  if constexpr (STAGED) for_each_chunk<STAGED>(table, c0, n, sweep);
  else
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) sweep(read_entry(&table[c0 + adam_chunk_of(i, n, order)]), 0);
}

// ---- LAMB -------------------------------------------------------------------------
//
// LAMB (You et al. 2020, the optimizer the paper weighs Adam against in Sec. 2.2 and
// Sec. 5) keeps Adam's moments and direction u = mhat / (sqrt(vhat) + eps) + wd p, and
// scales each tensor's step by the trust ratio ||p|| / ||u||.  The ratio needs sums
// over whole tensors, so the sweep is split in two, over a tensor-major chunk table:
//   k_lamb_moments : g, p, m, v -> m, v; per-chunk sums of p^2 and u^2
//   k_lamb_trust   : per tensor, the sums in chunk order (fp64) -> ratio, -lr * ratio
//   k_lamb_update  : p, m, v -> p + (-lr ratio) u, u recomputed from the stored moments
// (recomputing u costs the same 16 B/element as storing and re-reading it would, and
// leaves the gradients alone).  Both stages evaluate u with the same correctly rounded
// operations on the same fp32 inputs, so the u that is applied is the u that was measured.

// Combines per-lane values of the four wavefronts in a fixed order; the result is valid in thread 0.
__device__ __forceinline__ double block_sum(double x, double* s_w) {
  x = wave_sum(x);
  if ((threadIdx.x & 63u) == 0) s_w[threadIdx.x >> 6] = x;
  __syncthreads();
  return ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
}

// LAMB's first sweep over one chunk: moments updated and stored, the chunk's sums of
// p^2 and u^2 written to out[0], out[1] (fp64; per lane 4 * chunk_elems / 1024 squares
// are added in fp32 first; AGENT: by stores that another workgroup of the launch can read back).  coef != 1 only behind clipping; WB: the scaled gradient,
// rounded to its storage type, also replaces g.  GNT: whether g streams (it does not
// when the squared-norm pass has just read it and it is still cached).
template <int GDT, bool FUSED, bool WB, bool GNT, bool KEEP = false, bool AGENT = false>
__device__ __forceinline__ void lamb_moments_chunk(const Entry& en, float coef, const AdamK& k, double* s_pp,
                                                   double* s_uu, double* __restrict__ out) {
  typedef Grad<GDT> G;
  constexpr uint32_t gsize = sizeof(typename G::elem);
  const uint32_t tid = threadIdx.x;
  const bool wb = WB && coef != 1.f;
  const float wd = chunk_wd(en, k);
  const uint32_t len = en.len;
  uint32_t head = vector_head(len, en.p, en.m, en.v);
  // gradients that do not lie at the parameters' alignment, in plans that allow it (see kChunkLambByElement)
  if constexpr (!AGENT)
    if ((((en.p ^ en.m) | (en.p ^ en.v)) & 15u) == 0 && ((en.g + (uint64_t)head * gsize) & (4u * gsize - 1u)) != 0 &&
        (en.flags & (FUSED ? kChunkClipLambByElement : kChunkLambByElement)) != 0u)
      head = len;
  const uint32_t nvec = (len - head) / 4u;
  const uint32_t tail0 = head + nvec * 4u;
  void* gv = reinterpret_cast<void*>(en.g + (uint64_t)head * gsize);
  const f32x4* pv = reinterpret_cast<const f32x4*>(en.p + (uint64_t)head * 4u);
  f32x4* mv = reinterpret_cast<f32x4*>(en.m + (uint64_t)head * 4u);
  f32x4* vv = reinterpret_cast<f32x4*>(en.v + (uint64_t)head * 4u);
  float pp = 0.f, uu = 0.f;
  for (uint32_t j = tid; j < nvec; j += kBlock) {
    f32x4 g = G::template load4<GNT>(gv, j), p = ldv<true>(pv + j), m = ldv<true>(mv + j), v = ldv<true>(vv + j);
    loads_issued();
    if constexpr (FUSED) g = g * coef;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float mi = m[i], vi = v[i];
      adam_moments(g[i], mi, vi, k);
      const float u = adam_direction(p[i], mi, vi, k, wd);
      pp = __fmaf_rn(p[i], p[i], pp), uu = __fmaf_rn(u, u, uu);
      m[i] = mi, v[i] = vi;
    }
    stv<!KEEP>(mv + j, m), stv<!KEEP>(vv + j, v);
    if (wb) G::template store4<GNT>(gv, j, g);
  }
  void* gbase = reinterpret_cast<void*>(en.g);
  const BCA_GLOBAL float* p1 = as_global(reinterpret_cast<const float*>(en.p));
  BCA_GLOBAL float* m1 = as_global(reinterpret_cast<float*>(en.m));
  BCA_GLOBAL float* v1 = as_global(reinterpret_cast<float*>(en.v));
  for (uint32_t r = tid; r < head + (len - tail0); r += kBlock) {
    const uint32_t i = r < head ? r : tail0 + (r - head);
    float g = G::load1(gbase, i), m = m1[i], v = v1[i];
    const float p = p1[i];
    if constexpr (FUSED) g = g * coef;
    adam_moments(g, m, v, k);
    const float u = adam_direction(p, m, v, k, wd);
    pp = __fmaf_rn(p, p, pp), uu = __fmaf_rn(u, u, uu);
    m1[i] = m, v1[i] = v;
    if (wb) G::store1(gbase, i, g);
  }
  const double tpp = block_sum((double)pp, s_pp), tuu = block_sum((double)uu, s_uu);
  if (tid == 0) {
    if constexpr (AGENT) {
      __hip_atomic_store(&out[0], tpp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&out[1], tuu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      out[0] = tpp, out[1] = tuu;
    }
  }
}

template <int GDT, bool FUSED, bool WB, bool KEEP>
__global__ __launch_bounds__(kBlock) void k_lamb_moments(const Chunk* __restrict__ table, uint32_t n,
                                                          const float* __restrict__ coefs,
                                                          double* __restrict__ sums, const AdamK ka) {
  __shared__ double s_pp[kWaves], s_uu[kWaves];
  const AdamK k = resolve(ka);
  for (uint32_t ci = blockIdx.x; ci < n; ci += gridDim.x) {
    const Entry en = read_entry(&table[ci]);
    float coef = 1.f;
    if constexpr (FUSED) coef = coefs[en.bucket];
    lamb_moments_chunk<GDT, FUSED, WB, true, KEEP>(en, coef, k, s_pp, s_uu, sums + (uint64_t)ci * 2u);
    __syncthreads();  // s_pp / s_uu are reused by the next chunk
  }
}

// One workgroup of 1024 threads per tensor: the chunk sums strided over the threads (two
// independent accumulators each, the word embedding alone has 30 K chunks), butterfly per
// wavefront, the sixteen wavefronts in index order; then trust = ||p|| / ||u||, or 1
// where either norm is zero and the quotient means nothing; scale = -lr * trust in fp64,
// rounded once.  The order is fixed, so the ratios are reproducible.
constexpr uint32_t kTrustBlock = 1024;
__global__ __launch_bounds__(kTrustBlock) void k_lamb_trust(const double* __restrict__ sums,
                                                             const uint32_t* __restrict__ tensor_off, const AdamK ka,
                                                             float* __restrict__ trust, float* __restrict__ scale) {
  __shared__ double s_pp[kTrustBlock / 64], s_uu[kTrustBlock / 64];
  const double lr = resolve(ka).lr;
  const uint32_t t = blockIdx.x, lo = tensor_off[t], hi = tensor_off[t + 1];
  double pp0 = 0.0, uu0 = 0.0, pp1 = 0.0, uu1 = 0.0;
  uint32_t c = lo + threadIdx.x;
  for (; c + kTrustBlock < hi; c += 2u * kTrustBlock) {
    pp0 += sums[(uint64_t)c * 2u], uu0 += sums[(uint64_t)c * 2u + 1u];
    pp1 += sums[(uint64_t)(c + kTrustBlock) * 2u], uu1 += sums[(uint64_t)(c + kTrustBlock) * 2u + 1u];
  }
  if (c < hi) pp0 += sums[(uint64_t)c * 2u], uu0 += sums[(uint64_t)c * 2u + 1u];
  const double pp = wave_sum(pp0 + pp1), uu = wave_sum(uu0 + uu1);
  if ((threadIdx.x & 63u) == 0) s_pp[threadIdx.x >> 6] = pp, s_uu[threadIdx.x >> 6] = uu;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tpp = 0.0, tuu = 0.0;
    for (uint32_t w = 0; w < kTrustBlock / 64; ++w) tpp += s_pp[w], tuu += s_uu[w];
    const double pn = sqrt(tpp), un = sqrt(tuu);
    const double r = (pn > 0.0 && un > 0.0) ? pn / un : 1.0;
    trust[t] = (float)r;
    scale[t] = (float)(-lr * r);
  }
}

// The second sweep over one chunk: p + sc * u, u recomputed from the stored moments.
__device__ __forceinline__ void lamb_update_chunk(const Entry& en, float sc, const AdamK& k) {
  const uint32_t tid = threadIdx.x;
  const float wd = chunk_wd(en, k);
  const uint32_t len = en.len;
  const uint32_t head = vector_head(len, en.p, en.m, en.v);
  const uint32_t nvec = (len - head) / 4u;
  const uint32_t tail0 = head + nvec * 4u;
  f32x4* pv = reinterpret_cast<f32x4*>(en.p + (uint64_t)head * 4u);
  const f32x4* mv = reinterpret_cast<const f32x4*>(en.m + (uint64_t)head * 4u);
  const f32x4* vv = reinterpret_cast<const f32x4*>(en.v + (uint64_t)head * 4u);
  for (uint32_t j = tid; j < nvec; j += kBlock) {
    f32x4 p = ldv<true>(pv + j);
    const f32x4 m = ldv<true>(mv + j), v = ldv<true>(vv + j);
    loads_issued();
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = __fmaf_rn(sc, adam_direction(p[i], m[i], v[i], k, wd), p[i]);
    stv<true>(pv + j, p);
  }
  BCA_GLOBAL float* p1 = as_global(reinterpret_cast<float*>(en.p));
  const BCA_GLOBAL float* m1 = as_global(reinterpret_cast<const float*>(en.m));
  const BCA_GLOBAL float* v1 = as_global(reinterpret_cast<const float*>(en.v));
  for (uint32_t r = tid; r < head + (len - tail0); r += kBlock) {
    const uint32_t i = r < head ? r : tail0 + (r - head);
    p1[i] = __fmaf_rn(sc, adam_direction(p1[i], m1[i], v1[i], k, wd), p1[i]);
  }
}

__global__ __launch_bounds__(kBlock) void k_lamb_update(const Chunk* __restrict__ table, uint32_t n,
                                                         const float* __restrict__ scale, const AdamK ka) {
  const AdamK k = resolve(ka);
  for (uint32_t ci = blockIdx.x; ci < n; ci += gridDim.x) {
    const Entry en = read_entry(&table[ci]);
    lamb_update_chunk(en, scale[en.tensor], k);
  }
}

// ---- the whole fused step in one launch ----------------------------------------------
//
// Work items (one per workgroup) are listed by the host in an order that
// pipelines bucket groups:  N(g0) N(g1) A(g0) N(g2) A(g1) ... A(last), where N(g)
// are the squared-norm chunks of group g's buckets and A(g) the Adam chunks.  A
// group's gradients are read by N(g), stay in the Infinity Cache (everything
// else streams past it with non-temporal accesses), and are read again by A(g)
// one group later, so HBM sees the gradients once.
//
// An Adam item needs its bucket's coefficient; it waits on that bucket's ready
// word, which is set by whichever squared-norm workgroup of the bucket finishes
// last (it adds the bucket's partials in the fixed order of k_finalize, so
// results do not depend on who that is).  All squared-norm items of a bucket
// precede its Adam items in the list and never wait themselves.
//
// Which workgroup takes which item:
//  * default: item = workgroup index.  The hardware has been seen to start the
//    workgroups of a grid in index order within each XCD, so that everything an
//    Adam item waits for has been started before it; that is what makes the
//    pipeline fast, but nothing below depends on it for its result.
//  * TICKETS: eight atomic counters, one per XCD; item 8 t + y is the t-th item
//    of list y.  A workgroup draws from its own XCD's list and moves to the next
//    list when that one is used up.  Each list is thus started strictly in order
//    by running workgroups, whatever the dispatcher does.
//
// Every wait is bounded: after StepState::spin_limit polls the item gives up, files
// its index in the skipped list, raises the abort word (every other waiter then
// gives up at its next look) and BCA_STATUS_TIMEOUT, and its workgroup ends, which
// frees the slot for whatever it was waiting for.  Squared-norm items never wait, so
// by the end of the launch every bucket's coefficient exists, and the finish kernel
// that follows every such launch on the stream carries out the skipped items with
// the same code.  The call's result is therefore complete and bit-identical whatever
// the order in which workgroups were started; an expired wait only costs time.
//
// Per-call state needs no kernel in front of the launch: the last squared-norm item of a
// bucket zeroes that bucket's arrival counter, and the finish kernel hands the collected
// status bits to the caller, clears the abort word, the skipped count and the tickets and
// moves the epoch on, so that the state is ready for the next call on the plan.
//
// Small plans do without the finish kernel (SELF): the workgroup whose item is decided last
// carries out the skipped items and readies the state.

// Waits until this wavefront's outstanding vector-memory operations have completed (stores
// included: gfx9-family stores are counted by vmcnt until they are acknowledged).
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ uint32_t ctl_load(const uint32_t* w) {
  return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ctl_store(uint32_t* w, uint32_t x) {
  __hip_atomic_store(w, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ctl_or(uint32_t* w, uint32_t bits) {
  (void)__hip_atomic_fetch_or(w, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Shared memory of one k_step workgroup.
struct StepShared {
  uint32_t item;
  uint32_t flag;
  float coef;
  double w[kWaves];
  double pp[kWaves], uu[kWaves];  // LAMB: block sums of p^2 and u^2
};

// Waits (bounded) for bucket b's ready word of this epoch.  Returns true with the
// bucket's coefficient in sh.coef; false when the wait expired, after filing `self`
// (the item's index in the apply table) for the finish kernel.
__device__ __forceinline__ bool wait_for_bucket(const StepState& st, uint32_t b, uint32_t epoch, uint32_t self,
                                                StepShared& sh) {
  if (threadIdx.x == 0) {
    // ready word: (epoch << 32) | bits of the coefficient
    unsigned long long r = 0;
    uint32_t polls = 0;
    for (;;) {
      r = __hip_atomic_load(&st.ready[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((uint32_t)(r >> 32) == epoch || ++polls > st.spin_limit) break;
      // once one wait has expired every other waiter gives up at its next look
      if ((polls & 63u) == 0 && ctl_load(&st.ctl[kCtlAbort]) != 0u) break;
      __builtin_amdgcn_s_sleep(8);
    }
    const bool ok = (uint32_t)(r >> 32) == epoch;
    sh.flag = ok ? 1u : 0u;
    sh.coef = __uint_as_float((uint32_t)r);
    if (polls != 0u) {  // statistics (bca_plan_wait_stats); an item that never waited does not come here
      uint32_t* slot = &st.ctl[kCtlStats + 32u * (blockIdx.x % kStatSlots)];
      atomicAdd(slot, 1u);
      atomicAdd(reinterpret_cast<unsigned long long*>(slot + 2), (unsigned long long)polls);
    }
    if (!ok) {
      ctl_store(&st.ctl[kCtlAbort], 1u);
      ctl_or(&st.ctl[kCtlStatus], BCA_STATUS_TIMEOUT);
      // every item is filed at most once, so the list cannot overflow unless an earlier call on the plan was
      // cut short between its two launches; then the item is reported lost rather than written out of bounds
      const uint32_t slot = atomicAdd(&st.ctl[kCtlSkipped], 1u);
      if (slot < st.skipped_cap) ctl_store(&st.skipped[slot], self);  // read by whoever finishes the call
      else ctl_or(&st.ctl[kCtlStatus], BCA_STATUS_INCOMPLETE);
    }
  }
  __syncthreads();
  return sh.flag != 0u;
}

// A thread's share of the sum of partials [lo, hi) of a bucket, in k_finalize's order: thread t adds partials lo + t, lo + t + 256, ...
// one after the other.  The loads are issued eight at a time before the first addition (this workgroup is the one everybody else is
// waiting for, and an agent-scope load that misses every cache takes a microsecond or two); a slot past the end adds +0.0, which
// leaves a sum of squares as it is.
__device__ __forceinline__ double agent_partials(const StepState& st, uint64_t lo, uint64_t hi) {
  double s = 0.0;
  for (uint64_t i = lo + threadIdx.x; i < hi; i += 8u * kBlock) {
    double part[8];
#pragma unroll
    for (uint32_t q = 0; q < 8u; ++q) {
      const uint64_t j = i + (uint64_t)q * kBlock;
      part[q] = j < hi ? __hip_atomic_load(&st.partials[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
    }
#pragma unroll
    for (uint32_t q = 0; q < 8u; ++q) s += part[q];
  }
  return s;
}

// Norm and coefficient of bucket b from its sum of squares, and its ready word (thread 0).
__device__ __forceinline__ void publish_bucket(const StepState& st, uint32_t b, double tot, float threshold, uint32_t epoch,
                                               float* __restrict__ norms, float* __restrict__ coefs) {
  const float norm = (float)sqrt(tot);
  int32_t bst = 0;
  const float coef = clip_coef(norm, threshold, bst);
  norms[b] = norm;
  coefs[b] = coef;
  if (bst) ctl_or(&st.ctl[kCtlStatus], (uint32_t)bst);
  // The coefficient travels inside the ready word, so a waiter needs nothing else that this item wrote.
  const unsigned long long word = ((unsigned long long)epoch << 32) | (unsigned long long)__float_as_uint(coef);
  __hip_atomic_store(&st.ready[b], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The tail of every squared-norm item (kItemNorm, or kItemEmpty, the stand-in for a bucket without elements).  The last workgroup of a
// bucket to get here adds the bucket's partials in the fixed order of k_finalize, writes norm and coefficient and publishes the ready word.
//
// Why the last arriver sees every partial.  A partial is written by an agent-scope
// atomic store, which on this target is a write-through store that is acknowledged
// once it has reached the level at which the whole device is coherent; the storing
// wavefront then waits for that acknowledgement (vmcnt(0)) *before* the workgroup
// barrier, so when thread 0 counts the workgroup's arrival (after the barrier) all
// four partials of the chunk are visible to any agent-scope load.  Read-modify-write
// operations on arrived[b] are totally ordered; the workgroup whose increment makes the
// count complete therefore runs after every other arrival, hence after every partial
// of the bucket became visible, and its own loads of the partials (agent scope: they
// do not hit lines a per-XCD L2 may still hold from an earlier call) are issued only
// after its increment has returned.  A workgroup-scope release fence would not do: on
// this target it does not wait for vector stores, so the arrival could be counted
// while a partial is still on its way.
//
// `stored` chunks' partials of bucket b have just been written by this
// workgroup (0: a bucket without elements, nothing to count): waits for them, counts the arrival, and if
// this workgroup completes the bucket, finalizes it and publishes the ready word.
__device__ __forceinline__ void norm_arrive(const StepState& st, uint32_t b, uint32_t stored, uint32_t epoch,
                                            const float* __restrict__ thresholds, float* __restrict__ norms,
                                            float* __restrict__ coefs, StepShared& sh) {
  const uint32_t tid = threadIdx.x;
  if (stored != 0) {
    wait_vmem();      // the partials have been acknowledged ...
    __syncthreads();  // ... for every wavefront of the workgroup
    if (tid == 0) {
      const uint32_t total = st.norm_bucket_off[b + 1] - st.norm_bucket_off[b];
      const uint32_t old = atomicAdd(&st.arrived[b], stored);
      const bool last = (old + stored == total);
      // nobody else touches the counter again in this call: leave it at zero for the next one
      if (last) ctl_store(&st.arrived[b], 0u);
      sh.flag = last ? 1u : 0u;
    }
    __syncthreads();
    if (!sh.flag) return;
  }
  const uint64_t lo = (uint64_t)st.norm_bucket_off[b] * kWaves, hi = (uint64_t)st.norm_bucket_off[b + 1] * kWaves;
  const double s = wave_sum(agent_partials(st, lo, hi));
  if ((tid & 63u) == 0) sh.w[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) publish_bucket(st, b, ((sh.w[0] + sh.w[1]) + sh.w[2]) + sh.w[3], thresholds[b], epoch, norms, coefs);
}

__device__ __forceinline__ void store_partial(const StepState& st, uint32_t chunk, double ws) {
  if ((threadIdx.x & 63u) == 0)
    __hip_atomic_store(&st.partials[(uint64_t)chunk * kWaves + (threadIdx.x >> 6)], ws, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// All squared norms of a small plan in one launch, one workgroup per chunk, for calls that need every norm before any update (whole-gradient
// clipping, the step that is skipped on Inf or NaN).  Partials are exchanged as norm_arrive does it, for its reasons; whichever workgroup
// completes a bucket adds its partials up in k_finalize's order, and the one that completes the last bucket does what k_whole_coef does, hands
// over the status bits and leaves the counters at zero.  Two launches fewer than k_sqnorm, k_finalize and k_whole_coef (one without
// whole-gradient clipping), and the same bits; kOneLaunchNormChunks says where it pays.  n_filled: buckets with elements.
template <int GDT>
__global__ __launch_bounds__(kBlock) void k_norms(StepState st, uint32_t n, uint32_t n_buckets, uint32_t n_filled, bool whole,
                                                   const float* __restrict__ thresholds, float* __restrict__ norms,
                                                   float* __restrict__ coefs, double* __restrict__ bucket_sq, int32_t* status) {
  __shared__ double s_w[kWaves];
  __shared__ uint32_t s_last;
  __shared__ float s_coef;
  const uint32_t tid = threadIdx.x;
  if (blockIdx.x == 0) {  // buckets without elements
    int32_t bst = 0;
    for (uint32_t b = tid; b < n_buckets; b += kBlock) {
      if (st.norm_bucket_off[b] == st.norm_bucket_off[b + 1]) {
        norms[b] = 0.f;
        __hip_atomic_store(&bucket_sq[b], 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!whole) coefs[b] = clip_coef(0.f, thresholds[b], bst);
      }
    }
    if (bst != 0) ctl_or(&st.ctl[kCtlNormsStatus], (uint32_t)bst);
  }
  if (blockIdx.x < n) {
    const Entry en = read_entry(&st.norm_tab[blockIdx.x]);
    const uint32_t b = en.bucket, lo = st.norm_bucket_off[b], hi = st.norm_bucket_off[b + 1];
    store_partial(st, blockIdx.x, sqnorm_chunk<GDT, true, 16>(en));
    wait_vmem();      // the partials (and what has been stored above) have been acknowledged ...
    __syncthreads();  // ... for every wavefront of the workgroup
    if (tid == 0) {
      const bool last = atomicAdd(&st.arrived[b], 1u) + 1u == hi - lo;
      if (last) ctl_store(&st.arrived[b], 0u);  // left at zero for the next call
      s_last = last ? 1u : 0u;
    }
    __syncthreads();
    if (s_last == 0u) return;
    const double s = wave_sum(agent_partials(st, (uint64_t)lo * kWaves, (uint64_t)hi * kWaves));
    if ((tid & 63u) == 0) s_w[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
      const double tot = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
      const float norm = (float)sqrt(tot);
      int32_t bst = 0;
      norms[b] = norm;
      if (whole) __hip_atomic_store(&bucket_sq[b], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else coefs[b] = clip_coef(norm, thresholds[b], bst);
      if (bst != 0) ctl_or(&st.ctl[kCtlNormsStatus], (uint32_t)bst);
      wait_vmem();  // the sum and the bits have arrived before the bucket is counted
      const bool last = atomicAdd(&st.ctl[kCtlNormsDone], 1u) + 1u == n_filled;
      if (last) ctl_store(&st.ctl[kCtlNormsDone], 0u);
      s_last = last ? 1u : 0u;
    }
    __syncthreads();
    if (s_last == 0u) return;
  } else {  // a plan without elements: this is the only workgroup
    wait_vmem();
    __syncthreads();
  }
  if (whole) {
    double s = 0.0;
    for (uint32_t b = tid; b < n_buckets; b += kBlock)
      s += __hip_atomic_load(&bucket_sq[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s = wave_sum(s);
    if ((tid & 63u) == 0) s_w[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
      const float norm = (float)sqrt(((s_w[0] + s_w[1]) + s_w[2]) + s_w[3]);
      int32_t bst = 0;
      s_coef = clip_coef(norm, thresholds[0], bst);
      norms[n_buckets] = norm;
      if (bst != 0) ctl_or(&st.ctl[kCtlNormsStatus], (uint32_t)bst);
    }
    __syncthreads();
    for (uint32_t b = tid; b < n_buckets; b += kBlock) coefs[b] = s_coef;
  }
  if (tid == 0) {
    wait_vmem();
    *status = (int32_t)ctl_load(&st.ctl[kCtlNormsStatus]);
    ctl_store(&st.ctl[kCtlNormsStatus], 0u);
  }
}

// A squared-norm item of k_step: `count` consecutive chunks of the norm table (all of one bucket), first
// chunk idx; or (kItemEmpty) the stand-in for bucket idx, which has no elements.  A chunk's partials are the
// same whichever item it was part of.
template <int GDT>
__device__ __forceinline__ void norm_item(const StepState& st, uint32_t kind, uint32_t idx, uint32_t count,
                                          uint32_t epoch, const float* __restrict__ thresholds,
                                          float* __restrict__ norms, float* __restrict__ coefs, StepShared& sh) {
  if (kind != kItemNorm) {
    norm_arrive(st, idx, 0u, epoch, thresholds, norms, coefs, sh);
    return;
  }
  uint32_t b = 0;
  for (uint32_t c = idx; c < idx + count; ++c) {
    const Entry en = read_entry(&st.norm_tab[c]);
    b = en.bucket;
    // not ODD: k_step would need 70 registers instead of 55, and lose an eighth of its wavefronts wherever the gradients lie
    store_partial(st, c, sqnorm_chunk<GDT, false, 8, false>(en));
  }
  norm_arrive(st, b, count, epoch, thresholds, norms, coefs, sh);
}

// A squared-norm item where the launch is a chain of round trips to memory and little else (EARLY).  What finalizing the bucket takes is
// fetched beside the gradients, and a bucket of one chunk needs no exchange with other workgroups.  Others exchange their partials as in
// norm_arrive, for whose reasons the stores, the wait, the barrier and the count come in this order.
template <int GDT>
__device__ __forceinline__ void norm_item_short(const StepState& st, uint32_t idx, uint32_t count, uint32_t epoch,
                                                const float* __restrict__ thresholds, float* __restrict__ norms,
                                                float* __restrict__ coefs, StepShared& sh) {
  const uint32_t tid = threadIdx.x;
  Entry en = read_entry(&st.norm_tab[idx]);
  const uint32_t b = en.bucket;
  const uint32_t lo = st.norm_bucket_off[b], total = st.norm_bucket_off[b + 1] - lo;
  const float threshold = thresholds[b];
  if (total == 1u) {
    const double ws = sqnorm_chunk<GDT, false, 8, false>(en);
    if ((tid & 63u) == 0) sh.w[tid >> 6] = ws;
    __syncthreads();
    // as four partials in the first four lanes of a wavefront are added up
    if (tid == 0) publish_bucket(st, b, (sh.w[0] + sh.w[2]) + (sh.w[1] + sh.w[3]), threshold, epoch, norms, coefs);
    return;
  }
  for (uint32_t c = idx;;) {
    store_partial(st, c, sqnorm_chunk<GDT, false, 8, false>(en));
    if (++c == idx + count) break;
    en = read_entry(&st.norm_tab[c]);
  }
  wait_vmem();      // the partials have been acknowledged ...
  __syncthreads();  // ... for every wavefront of the workgroup: only now is the arrival counted
  if (tid == 0) {
    const bool last = atomicAdd(&st.arrived[b], count) + count == total;
    if (last) ctl_store(&st.arrived[b], 0u);
    sh.flag = last ? 1u : 0u;
  }
  __syncthreads();
  if (!sh.flag) return;
  const double s = wave_sum(agent_partials(st, (uint64_t)lo * kWaves, (uint64_t)(lo + total) * kWaves));
  if ((tid & 63u) == 0) sh.w[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) publish_bucket(st, b, ((sh.w[0] + sh.w[1]) + sh.w[2]) + sh.w[3], threshold, epoch, norms, coefs);
}

// What the items that wait for a coefficient do with it.
constexpr int kModeAdam = 0, kModeLamb = 1;

template <int GDT, bool WB, uint32_t U, int MODE>
__device__ __forceinline__ void apply_item(const StepState& st, const Entry& en, uint32_t idx, float coef,
                                           const AdamK& k, StepShared& sh) {
  if constexpr (MODE == kModeLamb)
    // LAMB's first sweep in place of Adam: moments and the chunk's two sums, filed under the chunk's place in
    // the tensor-major order; the trust ratio and the parameter update follow as launches of their own.
    lamb_moments_chunk<GDT, true, WB, false>(en, coef, k, sh.pp, sh.uu, st.lamb_sums + (uint64_t)st.apply_to_lamb[idx] * 2u);
  else
    adam_chunk<GDT, true, WB, U, false>(en, coef, k);
}

// Carries out the items whose wait expired (none, as a rule; one after the other if there are any -- an expired wait has
// cost about a second already), with the coefficient their bucket's ready word holds by now.  Returns status bits.
template <int GDT, bool WB, uint32_t U, int MODE>
__device__ __forceinline__ uint32_t finish_items(const StepState& st, uint32_t epoch, const AdamK& ka, StepShared& sh) {
  const uint32_t n_skipped = min(ctl_load(&st.ctl[kCtlSkipped]), st.skipped_cap);
  uint32_t bits = 0;
  if (n_skipped != 0) {
    const AdamK k = resolve(ka);
    for (uint32_t i = 0; i < n_skipped; ++i) {
      const uint32_t idx = ctl_load(&st.skipped[i]);
      const Entry en = read_entry(&st.apply_tab[idx]);
      const unsigned long long r = __hip_atomic_load(&st.ready[en.bucket], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((uint32_t)(r >> 32) != epoch) {  // cannot happen: squared-norm items never wait
        bits |= BCA_STATUS_INCOMPLETE;
        continue;
      }
      apply_item<GDT, WB, U, MODE>(st, en, idx, __uint_as_float((uint32_t)r), k, sh);
      __syncthreads();  // LAMB: sh.pp / sh.uu are reused by the next item
    }
  }
  return bits;
}

// Hands the status bits collected during the call to the caller and resets the per-call state, epoch included (thread 0).
__device__ __forceinline__ void finish_state(const StepState& st, uint32_t epoch, uint32_t collected, int32_t* status) {
  if (status != nullptr) *status = (int32_t)collected;
  // without a status word a lost item is reported by the plan's next pipelined call that has one
  ctl_store(&st.ctl[kCtlStatus], status != nullptr ? 0u : collected & (uint32_t)BCA_STATUS_INCOMPLETE);
  ctl_store(&st.ctl[kCtlSkipped], 0u);
  ctl_store(&st.ctl[kCtlAbort], 0u);
  for (uint32_t y = 0; y < 8u; ++y) ctl_store(&st.ctl[kCtlTicket + 32u * y], 0u);
  ctl_store(&st.ctl[kCtlEpoch], epoch + 1u == 0u ? 1u : epoch + 1u);
}

// SELF: a workgroup whose item is decided (its squared norms are published, or its wait has ended, one way or the other, with
// everything it has filed in place) counts itself in one of kDoneSlots words, so that no word sees more than a share of
// the increments (about 8 ns each, one after the other); those that complete a word count it in one more.  Launches of at most
// kFewItems count there at once, which is a round trip less at their end.  Thread 0 only.
__device__ __forceinline__ uint32_t count_done(const StepState& st, uint32_t n_work) {
  return atomicAdd(&st.ctl[kCtlDone + 32u * (n_work <= kFewItems ? (uint32_t)kDoneSlots : blockIdx.x % kDoneSlots)], 1u);
}
// Whether the workgroup that `count_done` gave `before` is the last of the launch.
__device__ __forceinline__ bool last_done(const StepState& st, uint32_t n_work, uint32_t before) {
  if (n_work <= kFewItems) {
    if (before + 1u != n_work) return false;
    ctl_store(&st.ctl[kCtlDone + 32u * kDoneSlots], 0u);
    return true;
  }
  const uint32_t slot = blockIdx.x % kDoneSlots;
  if (before + 1u != n_work / kDoneSlots + (slot < n_work % kDoneSlots ? 1u : 0u)) return false;
  ctl_store(&st.ctl[kCtlDone + 32u * slot], 0u);  // left at zero for the next call
  const uint32_t slots = n_work < kDoneSlots ? n_work : (uint32_t)kDoneSlots;
  if (atomicAdd(&st.ctl[kCtlDone + 32u * kDoneSlots], 1u) + 1u != slots) return false;
  ctl_store(&st.ctl[kCtlDone + 32u * kDoneSlots], 0u);
  return true;
}

// SELF: the launch needs no k_finish behind it.  Every workgroup is counted once its item is decided, and the one that
// completes the count does what k_finish would.  Adam items are counted when their wait has ended and before they store
// anything, so that the round trip is hidden behind the item itself.  That is early enough: the workgroup that completes the count
// touches nothing but the items that were filed, whose owners return without a store, and the call's state.
// EARLY: for lists with items that load before they wait (kItemEarly); eight workgroups a compute unit even so.
template <int GDT, bool WB, uint32_t U, bool TICKETS, bool LAMB, bool SELF = false, bool EARLY = SELF>
__global__ __launch_bounds__(kBlock, EARLY ? 8 : 1) void k_step(StepState st, const uint32_t* __restrict__ work, uint32_t n_work,
                                                  const float* __restrict__ thresholds, float* __restrict__ norms,
                                                  float* __restrict__ coefs, const AdamK ka, int32_t* status) {
  __shared__ StepShared sh;
  constexpr int MODE = LAMB ? kModeLamb : kModeAdam;
  uint32_t before = 0;  // SELF, thread 0: what count_done returned
  const AdamK k = resolve(ka);
  uint32_t ticket;
  if constexpr (TICKETS) {
    // Eight ticket counters, one per XCD: item 8 t + y is the t-th item of list y.  A
    // workgroup draws from its own XCD's list and moves on to the next list when that
    // one is used up, so every list is started strictly in order and every item is
    // taken by exactly one of the n_work workgroups.
    if (threadIdx.x == 0) {
      const uint32_t xcc = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7u;  // HW_REG_XCC_ID[3:0]
      uint32_t it = 0xffffffffu;
      for (uint32_t a = 0; a < 8u; ++a) {
        const uint32_t y = (xcc + a) & 7u;
        const uint32_t t = atomicAdd(&st.ctl[kCtlTicket + 32u * y], 1u);
        if ((uint64_t)t * 8u + y < n_work) {
          it = t * 8u + y;
          break;
        }
      }
      sh.item = it;
    }
    __syncthreads();
    ticket = sh.item;
  } else {
    ticket = blockIdx.x;
  }
  if (ticket >= n_work) return;
  const uint32_t epoch = st.ctl[kCtlEpoch];  // left by the previous call's finish kernel, constant during this launch
  const uint32_t item = work[ticket];
  const uint32_t kind = item >> 30;
  if (kind == kItemAdam) {
    const uint32_t idx = item & kItemIndex;
    const Entry en = read_entry(&st.apply_tab[idx]);
    if constexpr (EARLY) {
      const auto wait = [&] {
        const bool ready = wait_for_bucket(st, en.bucket, epoch, idx, sh);
        if constexpr (SELF) {
          if (threadIdx.x == 0) {
            if (!ready) wait_vmem();  // what the wait has filed has arrived
            before = count_done(st, n_work);  // not looked at before the item is done
          }
        }
        return ready;
      };
      if ((item & kItemEarly) != 0u && en.len == 4u * kBlock) adam_chunk_early<GDT, WB>(en, k, &sh.coef, wait);
      else if (wait()) apply_item<GDT, WB, U, MODE>(st, en, idx, sh.coef, k, sh);
    } else {
      if (wait_for_bucket(st, en.bucket, epoch, idx, sh)) apply_item<GDT, WB, U, MODE>(st, en, idx, sh.coef, k, sh);
    }
  } else {
    // squared-norm items carry their chunk count (1 .. 4) in bits 28..29
    if (EARLY && kind == kItemNorm)
      norm_item_short<GDT>(st, item & 0x0fffffffu, ((item >> 28) & 3u) + 1u, epoch, thresholds, norms, coefs, sh);
    else
      norm_item<GDT>(st, kind, item & 0x0fffffffu, ((item >> 28) & 3u) + 1u, epoch, thresholds, norms, coefs, sh);
    if constexpr (SELF) {
      if (threadIdx.x == 0) {
        wait_vmem();  // status bits and ready word have arrived
        before = count_done(st, n_work);
      }
    }
  }
  if constexpr (SELF) {
    if (threadIdx.x == 0) sh.item = last_done(st, n_work, before) ? 1u : 0u;
    __syncthreads();
    if (sh.item == 0u) return;
    const uint32_t skipped = ctl_load(&st.ctl[kCtlSkipped]);
    uint32_t collected = ctl_load(&st.ctl[kCtlStatus]);
    if (skipped != 0u) {
      const uint32_t bits = finish_items<GDT, WB, U, MODE>(st, epoch, ka, sh);
      collected = ctl_load(&st.ctl[kCtlStatus]) | bits;
    }
    if (threadIdx.x == 0) finish_state(st, epoch, collected, status);
  }
}

// ---- LAMB in one pass over p, m, v -------------------------------------------------------
//
// LAMB's update needs its tensor's trust ratio, i.e. sums over the whole tensor, so that two sweeps read p, m and v
// twice: 40 bytes per element instead of the 28 that have to move.  The path is bound by what crosses the
// L2 / fabric boundary (about 6.9 TB/s whether HBM or the Infinity Cache answers), so a second read that hits the
// Infinity Cache is still paid for.  Here a workgroup keeps p and u of its item (12 chunks of 1 024 elements) on the chip, p and a third
// of u in registers, two thirds of u in LDS, stores the moments, and files the chunks' sums; the last workgroup of the tensor
// to get there derives the ratio and publishes -lr * ratio; the others wait for it and then write p.  Four
// workgroups per compute unit are resident (128 VGPRs, 33 KiB of LDS), 12.6 M elements in all.  A tensor's first
// workgroups wait until its last one is through, so the slots of half a tensor idle on average: larger items
// beat smaller ones although those stream better (335 M elements in tensors of 4 M: 8 chunks an item 1.83 ms, 12 with
// part of u in LDS 1.67; in tensors of 1 M: 1.58 and 1.64; two sweeps in runs 2.05).
// An item's chunks lie kLambStride apart where the tensor is long enough, and four of them are fetched at a time: BERT-Large lamb_step
// 1 748 us with items of consecutive chunks, two at a time; consecutive, four at a time 1 731; kLambStride apart, two 1 685, four 1 675;
// BERT-Base, fp16, behind clipping (tensors in allocations of their own, as everywhere here) 534, 533, 524 and 520.
//   BERT-Large, fp32: lamb_step 2085 us in two sweeps in runs, 1675 like this; BERT-Base, fp16, behind clipping 695 and 520.
//
// Sums are taken chunk by chunk and added in k_lamb_trust's order: results are those of the two sweeps bit for bit (where
// the gradients do not lie at the parameters' alignment, up to the grouping of the sums' fp32 terms).
//
// Tensors too large to be held (kLambHeldNum / kLambHeldDen; BERT's word embedding) are last in the list of lamb_step: their items store the
// moments cacheable and the tail kernel carries out their second sweep, most recent item first.  The end of such a tensor is held like a whole one
// (kLambEndsFrom).
//
// Waiting.  Items wait for the rest of their own tensor, which the work list keeps together and which is resident at
// once as a rule.  It need not be: another launch of this kind on the GPU may hold slots that it is waiting for, and
// they for it.  Every wait is therefore bounded, and short: an item that gives up files itself, raises a flag that makes
// other waiters give up at their next look, and ends; its moments and sums are stored, and the tail kernel, which
// follows every such launch, reads it again and updates p with the same arithmetic.  Behind clipping, items first
// wait for their bucket's coefficient, as in k_step; one that gives up there has done nothing, and is carried out (moments, sums,
// and the ratio of a tensor that it completes) by k_lamb_late, between the launch and its tail.

struct LambShared {
  StepShared step;
  double pp[kLambItemChunks][kWaves], uu[kLambItemChunks][kWaves];
  double tp[kTrustBlock / 64], tu[kTrustBlock / 64];
  uint32_t last;
  float scale;
  f32x4 u[2 * kLambItemChunks / 3][kBlock];
};

// k_lamb_trust for one tensor by a workgroup of 256 threads, each of whose wavefronts stands in for four of that kernel's
// sixteen; the sums may just have been written by other workgroups (agent scope).  Publishes the result.
__device__ __forceinline__ void tensor_ratio(const LambState& ls, uint32_t t, uint32_t lo, uint32_t hi, uint32_t epoch, double lr,
                                             LambShared& sh) {
  constexpr uint32_t Q = 2;  // of the four wavefronts that each one here stands in for, those handled at a time
  const uint32_t lane = threadIdx.x & 63u;
  // every workgroup of the tensor waits for this: a thread's loads are issued eight at a time
#pragma unroll
  for (uint32_t q0 = 0; q0 < kTrustBlock / kBlock; q0 += Q) {
    double pp0[Q] = {}, uu0[Q] = {}, pp1[Q] = {}, uu1[Q] = {};
    for (uint32_t base = lo + q0 * kBlock + threadIdx.x; base < hi; base += 2u * kTrustBlock) {
      double x[Q][4];
#pragma unroll
      for (uint32_t q = 0; q < Q; ++q) {
#pragma unroll
        for (uint32_t r = 0; r < 4u; ++r) {  // r & 1: which sum; r >> 1: which of the two accumulators
          const uint32_t c = base + q * kBlock + (r >> 1) * kTrustBlock;
          x[q][r] = 0.0;  // adds nothing to sums of squares
          if (c < hi) x[q][r] = __hip_atomic_load(&ls.sums[(uint64_t)c * 2u + (r & 1u)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
#pragma unroll
      for (uint32_t q = 0; q < Q; ++q) pp0[q] += x[q][0], uu0[q] += x[q][1], pp1[q] += x[q][2], uu1[q] += x[q][3];
    }
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {
      const double pp = wave_sum(pp0[q] + pp1[q]), uu = wave_sum(uu0[q] + uu1[q]);
      const uint32_t w = (q0 + q) * kWaves + (threadIdx.x >> 6);
      if (lane == 0) sh.tp[w] = pp, sh.tu[w] = uu;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tpp = 0.0, tuu = 0.0;
    for (uint32_t w = 0; w < kTrustBlock / 64; ++w) tpp += sh.tp[w], tuu += sh.tu[w];
    const double pn = sqrt(tpp), un = sqrt(tuu);
    const double r = (pn > 0.0 && un > 0.0) ? pn / un : 1.0;
    const float scale = (float)(-lr * r);
    const unsigned long long word = ((unsigned long long)epoch << 32) | (unsigned long long)__float_as_uint(scale);
    __hip_atomic_store(&ls.ready[t], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ls.trust[t] = (float)r;
    sh.scale = scale;
  }
}

// Thread 0's bounded wait for tensor t's ready word; false after filing `self` as late.
__device__ __forceinline__ bool wait_for_tensor(const StepState& st, const LambState& ls, uint32_t t, uint32_t epoch,
                                                uint32_t self, float* scale) {
  const uint32_t limit = min(st.spin_limit, kTrustSpinLimit);
  uint32_t polls = 0, aborted = 0;
  for (;;) {
    const unsigned long long r = __hip_atomic_load(&ls.ready[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // once one wait has expired nobody waits any more: items that start after that hardly hold their slots
    if (polls == 1u || (polls & 15u) == 15u) aborted = ctl_load(&st.ctl[kCtlLateAbort]);
    if ((uint32_t)(r >> 32) == epoch) {
      *scale = __uint_as_float((uint32_t)r);
      return true;
    }
    if (aborted != 0u || ++polls > limit) break;
    __builtin_amdgcn_s_sleep(16);
  }
  if (aborted == 0u) {  // the others have nothing to add
    ctl_store(&st.ctl[kCtlLateAbort], 1u);
    ctl_or(&st.ctl[kCtlStatus], BCA_STATUS_TIMEOUT);
  }
  const uint32_t slot = atomicAdd(&st.ctl[kCtlLate], 1u);
  if (slot < ls.n_items) ls.late[slot] = self;  // read by the tail kernel
  else ctl_or(&st.ctl[kCtlStatus], BCA_STATUS_INCOMPLETE);
  return false;
}

// Chunks of the tensor-major table from one chunk of an item to the next.
__device__ __forceinline__ uint32_t lamb_stride(uint32_t flags) { return (flags & kLambSpread) ? kLambStride : 1u; }

// One item: moments, sums, arrival, ratio; HOLD: then the wait and the update of a held item.
template <int GDT, bool CLIP, bool WB, bool HOLD>
__device__ __forceinline__ void lamb_item(const StepState& st, const LambState& ls, const LambItem* __restrict__ ip, uint32_t self,
                                          float coef, const AdamK& k, uint32_t epoch, LambShared& sh) {
  typedef Grad<GDT> G;
  constexpr uint32_t CH = kLambItemChunks, LD = 2 * CH / 3, B = WB ? 2 : 4;  // chunks; those whose u is in LDS; chunks loaded at a time (with write-back, four spill)
  constexpr bool GNT = !CLIP;  // behind clipping the gradients are in cache
  const uint32_t tid = threadIdx.x;
  const uint32_t first = ip->first, count = ip->count, t = ip->tensor, flags = ip->flags;
  const uint32_t items = ip->items, lo = ip->lo, hi = ip->hi, S = lamb_stride(flags);
  const bool regular = HOLD && (flags & kLambRegular) != 0u;
  const bool held = HOLD && (flags & (CLIP ? kLambHeld : kLambHeld | kLambHeldAlone)) != 0u;
  const float wd = (flags & kChunkNoDecay) ? 0.f : k.wd;
  f32x4 P[CH], U[CH - LD];
  if (regular) {
    const uint64_t ga = ip->g;
    f32x4* pv = reinterpret_cast<f32x4*>(ip->p);
    f32x4* mv = reinterpret_cast<f32x4*>(ip->m);
    f32x4* vv = reinterpret_cast<f32x4*>(ip->v);
    const bool keep = (flags & kLambKeep) != 0u && !held, wb = WB && coef != 1.f;
    // Whether the moments stay cached is decided out here, a sweep for each: with the two kinds of store in the arms of one branch the compiler
    // makes one store of them, without the streaming hint (BERT-Large lamb_step 1 848 us like that, 1 748 so; BERT-Base fp16 behind
    // the clip 568 and 534).  A plan of 8 M to 40 M elements that is stepped again with nothing in between found its moments cached like that, and does not
    // now: with all that has changed since, lamb_step fp32 11 M 61 -> 64 (in three tensors 62), 20 M 103 -> 108, 34 M 166 -> 180; with 1 GiB of other memory
    // swept in between, as a training step does, 73 -> 70, 122 -> 113, 198 -> 184.
    const auto sweep = [&](auto full, auto kept) {
    constexpr bool FULL = decltype(full)::value, KEEP = decltype(kept)::value;
#pragma unroll
    for (uint32_t j = 0; j < CH; ++j)  // p stays in registers anyway: all of it is fetched at once
      if (FULL || j < count) P[j] = ldv<true>(pv + j * S * kBlock + tid);
    loads_issued();
#pragma unroll
    for (uint32_t j = 0; j < CH; j += B) {
      if (FULL || j < count) {
        f32x4 g[B], m[B], v[B];
        float pp[B] = {}, uu[B] = {};
#pragma unroll
        for (uint32_t q = 0; q < B; ++q) {
          if (FULL || j + q < count) {
            g[q] = G::template load4<GNT>(reinterpret_cast<const void*>(ga + (uint64_t)((j + q) * S) * 1024u * sizeof(typename G::elem)), tid);
            m[q] = ldv<true>(mv + (j + q) * S * kBlock + tid);
            v[q] = ldv<true>(vv + (j + q) * S * kBlock + tid);
          }
        }
        loads_issued();
#pragma unroll
        for (uint32_t q = 0; q < B; ++q) {
          if (FULL || j + q < count) {
            if constexpr (CLIP) g[q] = g[q] * coef;
            f32x4 u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              float mi = m[q][i], vi = v[q][i];
              adam_moments(g[q][i], mi, vi, k);
              const float d = adam_direction(P[j + q][i], mi, vi, k, wd);
              pp[q] = __fmaf_rn(P[j + q][i], P[j + q][i], pp[q]), uu[q] = __fmaf_rn(d, d, uu[q]);
              m[q][i] = mi, v[q][i] = vi, u[i] = d;
            }
            stv<!KEEP>(mv + (j + q) * S * kBlock + tid, m[q]), stv<!KEEP>(vv + (j + q) * S * kBlock + tid, v[q]);
            if (wb)
              G::template store4<GNT>(reinterpret_cast<void*>(ga + (uint64_t)((j + q) * S) * 1024u * sizeof(typename G::elem)), tid, g[q]);
            if (j + q < LD) sh.u[j + q < LD ? j + q : 0][tid] = u;
            else U[j + q < LD ? 0 : j + q - LD] = u;
          }
        }
        // two chunks' sums at a time, each as wave_sum adds it up; rows 0 .. 3: p^2 of chunk q, of q + 1, u^2 of chunk q, of q + 1
#pragma unroll
        for (uint32_t q = 0; q < B; q += 2) {
          const double w = row_sum(add16(add32((double)pp[q], (double)uu[q]), add32((double)pp[q + 1], (double)uu[q + 1])));
          if ((tid & 15u) == 0) ((tid & 32u) ? sh.uu : sh.pp)[j + q + ((tid >> 4) & 1u)][tid >> 6] = w;
        }
        loads_issued();
      }
    }
    };
    // Full items that keep them have a sweep without tests per chunk too.  lamb_step, us, without / with it, other memory swept in between: 14 M and 6 x 4 Mi elements
    // 240.6 / 239.1, 2 x 15 M and 10 x 4 Mi 428.7 / 426.6, 31 M and 8 x 4 Mi 380.0 / 378.3; fp16 229.7 / 228.8, 408.7 / 407.0, 359.6 / 360.2.  Behind clipping it
    // gains nothing (464.1 / 464.5, 418.6 / 419.6).
    if (!CLIP && keep && count == CH) sweep(std::true_type{}, std::true_type{});
    else if (keep) sweep(std::false_type{}, std::true_type{});
    else if (count == CH) sweep(std::true_type{}, std::false_type{});
    else sweep(std::false_type{}, std::false_type{});
    __syncthreads();
    if (tid < 2u * count) {  // the four wavefronts' sums in index order; all in wavefront 0
      const uint32_t j = tid >> 1;
      const double* w = (tid & 1u) ? sh.uu[j] : sh.pp[j];
      __hip_atomic_store(&ls.sums[(uint64_t)(first + j * S) * 2u + (tid & 1u)], ((w[0] + w[1]) + w[2]) + w[3], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  } else {
    for (uint32_t j = 0; j < count; ++j) {
      lamb_moments_chunk<GDT, CLIP, WB, GNT, false, true>(read_entry(&ls.tab[first + j * S]), coef, k, sh.step.pp, sh.step.uu,
                                                          ls.sums + (uint64_t)(first + j * S) * 2u);
      __syncthreads();  // sh.step.pp / uu are reused by the next chunk
    }
  }
  // Arrival: the sums were stored by wavefront 0, which waits for their acknowledgement before it counts (see norm_arrive).
  if (tid < 64u) {
    wait_vmem();
    if (tid == 0) {
      const bool last = atomicAdd(&ls.arrived[t], 1u) + 1u == items;
      if (last) ctl_store(&ls.arrived[t], 0u);  // left at zero for the next call
      sh.last = last ? 1u : 0u;
    }
  }
  __syncthreads();
  const bool last = sh.last != 0u;
  if (last) tensor_ratio(ls, t, lo, hi, epoch, k.lr, sh);
  if (!held) return;
  if (!last && tid == 0) {
    float scale = 0.f;
    sh.step.flag = wait_for_tensor(st, ls, t, epoch, self, &scale) ? 1u : 0u;
    sh.scale = scale;
  }
  __syncthreads();
  if (!last && sh.step.flag == 0u) return;
  const float sc = sh.scale;
  if (regular) {
    f32x4* pv = reinterpret_cast<f32x4*>(ip->p);
#pragma unroll
    for (uint32_t j = 0; j < CH; ++j) {
      if (j < count) {
        const f32x4 u = j < LD ? sh.u[j < LD ? j : 0][tid] : U[j < LD ? 0 : j - LD];
        f32x4 x;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __fmaf_rn(sc, u[i], P[j][i]);
        stv<true>(pv + j * S * kBlock + tid, x);
      }
    }
  } else {
    // every thread reads back the elements that it has stored itself
    for (uint32_t j = 0; j < count; ++j) lamb_update_chunk(read_entry(&ls.tab[first + j * S]), sc, k);
  }
}

template <int GDT, bool CLIP, bool WB>
__global__ __launch_bounds__(kBlock, kLambResidentPerCu) void k_lamb(StepState st, LambState ls, const uint32_t* __restrict__ work,
                                                                     const float* __restrict__ thresholds, float* __restrict__ norms,
                                                                     float* __restrict__ coefs, const AdamK ka) {
  __shared__ LambShared sh;
  const AdamK k = resolve(ka);
  const uint32_t epoch = st.ctl[kCtlEpoch];  // left by the previous call, constant during this launch
  uint32_t i = blockIdx.x;  // without clipping the items are worked on in their own order
  float coef = 1.f;
  if constexpr (CLIP) {
    const uint32_t item = work[blockIdx.x], kind = item >> 30;
    i = item & 0x3fffffffu;
    if (kind != kItemAdam) {
      norm_item<GDT>(st, kind, item & 0x0fffffffu, ((item >> 28) & 3u) + 1u, epoch, thresholds, norms, coefs, sh.step);
      return;
    }
  }
  if constexpr (CLIP) {
    if (!wait_for_bucket(st, ls.items[i].bucket, epoch, i, sh.step)) return;
    coef = sh.step.coef;
  }
  lamb_item<GDT, CLIP, WB, true>(st, ls, &ls.items[i], i, coef, k, epoch, sh);
}

// Behind a clipping launch: the items that gave up waiting for their bucket's coefficient (none, as a rule), which
// exists by now.
template <int GDT, bool WB>
__global__ __launch_bounds__(kBlock) void k_lamb_late(StepState st, LambState ls, const AdamK ka) {
  __shared__ LambShared sh;
  // written by the launch before this one, so plain loads do (see k_lamb_tail)
  const uint32_t n = min(st.ctl[kCtlSkipped], st.skipped_cap);
  if (n == 0) return;
  const AdamK k = resolve(ka);
  const uint32_t epoch = st.ctl[kCtlEpoch];
  for (uint32_t q = blockIdx.x; q < n; q += gridDim.x) {
    const uint32_t i = st.skipped[q];
    const unsigned long long r = __hip_atomic_load(&st.ready[ls.items[i].bucket], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)(r >> 32) != epoch) {  // cannot happen: squared-norm items never wait
      if (threadIdx.x == 0) ctl_or(&st.ctl[kCtlStatus], BCA_STATUS_INCOMPLETE);
      continue;
    }
    lamb_item<GDT, true, WB, false>(st, ls, &ls.items[i], i, __uint_as_float((uint32_t)r), k, epoch, sh);
    __syncthreads();
  }
}

// Follows every k_lamb launch.  Workgroup w carries out the second sweep over the w-th chunk of the large tensors' items,
// the most recent one first (its moments are the likeliest to be in cache; a workgroup per item, chunk after chunk,
// takes 105 instead of 75 us over 31 M elements); the first kLambTailWorkers workgroups share the chunks of the items
// that gave up waiting, and the last of them to be done hands over the status bits and readies the state for the next
// call.  Tensors without elements get ratio 1.
// What it reads was written by earlier launches, so plain loads do; thousands of workgroups reading one word at agent scope
// would queue up behind it (10 ns each).  Only workers look at the epoch: it moves on once they are all done, which
// the other workgroups may still outlast.
__global__ __launch_bounds__(kBlock) void k_lamb_tail(StepState st, LambState ls, int32_t* status, const AdamK ka) {
  const uint32_t w = blockIdx.x, tid = threadIdx.x;
  const AdamK k = resolve(ka);
  const auto update = [&](uint32_t i, uint32_t from, uint32_t to) {  // chunks [from, to) of item i
    const LambItem* ip = &ls.items[i];
    const float sc = __uint_as_float((uint32_t)ls.ready[ip->tensor]);
    const uint32_t first = ip->first, S = lamb_stride(ip->flags), end = min(to, ip->count);
    for (uint32_t j = from; j < end; ++j) lamb_update_chunk(read_entry(&ls.tab[first + j * S]), sc, k);
  };
  const uint32_t back = w / kLambItemChunks, chunk = w % kLambItemChunks;
  if (back < ls.first_end - ls.first_large) update(ls.first_end - 1u - back, chunk, chunk + 1u);
  if (w >= kLambTailWorkers) return;
  const uint32_t n_late = min(st.ctl[kCtlLate], ls.n_items), n_skipped = min(st.ctl[kCtlSkipped], st.skipped_cap);
  // Without late items a few workers do.  The others find zeros here whether they look before the reset below or after it;
  // with late items there is no reset before all of them have been counted.
  const uint32_t workers = min(gridDim.x, n_late + n_skipped != 0u ? kLambTailWorkers : kLambTailFew);
  if (w >= workers) return;
  const uint32_t epoch = st.ctl[kCtlEpoch];
  for (uint32_t q = w; q < n_late * kLambItemChunks; q += workers)
    update(ls.late[q / kLambItemChunks], q % kLambItemChunks, q % kLambItemChunks + 1u);
  for (uint32_t q = w; q < n_skipped * kLambItemChunks; q += workers) {
    const uint32_t i = st.skipped[q / kLambItemChunks];
    if (ls.items[i].flags & kLambHeld) update(i, q % kLambItemChunks, q % kLambItemChunks + 1u);
  }
  for (uint32_t t = w * kBlock + tid; t < ls.n_tensors; t += workers * kBlock) {
    if (ls.items_of[t] == 0u) ls.trust[t] = 1.f;
    // cannot happen: every item's sums have been counted by now
    else if ((uint32_t)(ls.ready[t] >> 32) != epoch) ctl_or(&st.ctl[kCtlStatus], BCA_STATUS_INCOMPLETE);
  }
  wait_vmem();  // a status bit raised above has arrived before this worker is counted
  __syncthreads();
  if (tid == 0 && atomicAdd(&st.ctl[kCtlTailDone], 1u) + 1u == workers) {
    const uint32_t collected = ctl_load(&st.ctl[kCtlStatus]);
    if (status != nullptr) *status = (int32_t)collected;
    // as in finish_state; lamb_step has no status word
    ctl_store(&st.ctl[kCtlStatus], status != nullptr ? 0u : collected & (uint32_t)BCA_STATUS_INCOMPLETE);
    for (const uint32_t word : {kCtlSkipped, kCtlAbort, kCtlLate, kCtlLateAbort, kCtlTailDone}) ctl_store(&st.ctl[word], 0u);
    ctl_store(&st.ctl[kCtlEpoch], epoch + 1u == 0u ? 1u : epoch + 1u);
  }
}

// g <- coef * g over one chunk of the squared-norm cut.  A full chunk of kDefaultChunkNorm
// elements is fetched whole (every load in flight before the first store); anything else goes through scale_chunk.
// Element by element the stored value is the same either way.
template <int GDT>
__device__ __forceinline__ void scale_norm_chunk(const Entry& en, float coef) {
  typedef Grad<GDT> G;
  typedef typename G::wide wide;
  constexpr uint32_t R = kDefaultChunkNorm / (G::VE * kBlock);  // 128-bit pieces per lane: 16 (fp32) or 8 (16-bit types)
  if (en.len == kDefaultChunkNorm) {
    wide* gw = reinterpret_cast<wide*>(en.g);
    const uint32_t tid = threadIdx.x;
    wide x[R];
    if (G::VE == 8 && (en.g & 2u) != 0) {
      if constexpr (G::VE == 8) ld_odd<false>(x, gw + tid, kBlock);
    } else {
#pragma unroll
      for (uint32_t u = 0; u < R; ++u) x[u] = ldv<false>(gw + tid + u * kBlock);
    }
    loads_issued();
#pragma unroll
    for (uint32_t u = 0; u < R; ++u) {
      float f[G::VE];
      G::widen(x[u], f);
#pragma unroll
      for (uint32_t q = 0; q < G::VE; ++q) f[q] = f[q] * coef;
      stv<false>(gw + tid + u * kBlock, G::narrow(f));
    }
  } else {
    scale_chunk<GDT, 4, false>(en, coef);
  }
}

// The second of bucket_clip's two launches (the first is k_sqnorm over the range's chunks): one workgroup per
// squared-norm chunk.  Every workgroup adds up its bucket's partial sums itself, in k_finalize's order, so all of
// them arrive at the same norm and coefficient without exchanging anything (the partials of a 50 MiB bucket
// are 25 KB, read from L2 by every workgroup), and then scales its chunk; the workgroup of a bucket's first
// chunk also writes the bucket's norm and coefficient and ORs its status bits.  No workgroup waits for another.
// Workgroup 0 deals with the range's buckets that have no elements.
template <int GDT>
__global__ __launch_bounds__(kBlock) void k_clip_scale(const Chunk* __restrict__ norm_tab, uint32_t cn0, uint32_t n,
                                                        const uint32_t* __restrict__ bucket_chunk_off, uint32_t b0,
                                                        uint32_t b1, const double* __restrict__ partials,
                                                        const float* __restrict__ thresholds, float* __restrict__ norms,
                                                        float* __restrict__ coefs, int32_t* status) {
  __shared__ double s_w[kWaves];
  __shared__ float s_coef;
  const uint32_t tid = threadIdx.x;
  if (blockIdx.x == 0) {
    int32_t bst = 0;
    for (uint32_t b = b0 + tid; b < b1; b += kBlock) {
      if (bucket_chunk_off[b] == bucket_chunk_off[b + 1]) {
        norms[b] = 0.f;
        coefs[b] = clip_coef(0.f, thresholds[b], bst);
      }
    }
    if (bst != 0 && status != nullptr) atomicOr(status, bst);
  }
  if (blockIdx.x >= n) return;
  const uint32_t idx = cn0 + blockIdx.x;
  const Entry en = read_entry(&norm_tab[idx]);
  const uint32_t b = en.bucket;
  const double tot = sum_partials(partials, (uint64_t)bucket_chunk_off[b] * kWaves, (uint64_t)bucket_chunk_off[b + 1] * kWaves, s_w);
  if (tid == 0) {
    const float norm = (float)sqrt(tot);
    int32_t bst = 0;
    const float coef = clip_coef(norm, thresholds[b], bst);
    s_coef = coef;
    if (idx == bucket_chunk_off[b]) {
      norms[b] = norm;
      coefs[b] = coef;
      if (bst != 0 && status != nullptr) atomicOr(status, bst);
    }
  }
  __syncthreads();
  const float coef = s_coef;
  if (coef != 1.f) scale_norm_chunk<GDT>(en, coef);
}

// Follows every k_step launch that does not finish itself; ONE workgroup, so that it costs a launch and one round trip to
// memory when there is nothing to do.
template <int GDT, bool WB, uint32_t U, int MODE>
__global__ __launch_bounds__(kBlock) void k_finish(StepState st, int32_t* status, const AdamK ka) {
  __shared__ StepShared sh;
  const uint32_t epoch = ctl_load(&st.ctl[kCtlEpoch]);
  const uint32_t bits = finish_items<GDT, WB, U, MODE>(st, epoch, ka, sh);
  if (threadIdx.x == 0) finish_state(st, epoch, ctl_load(&st.ctl[kCtlStatus]) | bits, status);
}

// ---- clipping one contiguous bucket without a plan and without allocating ---------------
//
// For callers that cannot allocate (HIP graph capture, tight loops): the bucket is a
// pointer and a length, chunk bounds are computed from the chunk index instead of read
// from a table, and the partial sums live in a fixed array of this library's device
// image.  One launch for a bucket of one chunk; else two plain launches (squared norms; coefficient and scale; three for buckets of more than 16 Mi
// elements, whose coefficient gets a launch of its own) with the device functions
// of the plan-based path, so norm, coefficient and scaled gradients are those of
// bucket_clip on a one-tensor, one-bucket plan whose squared-norm chunk is kFlatChunkNorm.

constexpr uint32_t kFlatHeaderBytes = 256;  // one float: the coefficient of a large bucket, handed from its finalize launch to its scale launch
constexpr size_t kFlatScratchBytes = kFlatHeaderBytes + (size_t)(kFlatMaxElems / kFlatChunkNorm) * kWaves * sizeof(double);
static __device__ __align__(256) unsigned char scratch[kFlatScratchBytes];

// n <= kFlatMaxElems fits in 32 bits.  The length is a 32-bit minimum on purpose: written as a select on a 64-bit
// comparison, the compiler has been seen to take the wrong arm where it also branches on the length (the scalar unit
// has no 64-bit less-than; the select came out reading a condition code that nobody had set).
__device__ __forceinline__ Entry flat_entry(uint64_t g, uint32_t n, uint32_t chunk_elems, uint32_t gsize, uint32_t i) {
  const uint32_t first = i * chunk_elems;
  Entry e;
  e.g = g + (uint64_t)first * gsize, e.p = 0, e.m = 0, e.v = 0;
  e.len = min(n - first, chunk_elems);
  e.bucket = 0, e.tensor = 0, e.flags = 0;
  return e;
}

// A bucket of one chunk, clipped by one workgroup in one launch: `tab` is its entry in the squared-norm cut, or null for the n elements at g.
// Norm, coefficient and scaled gradients are those of the two launches (k_finalize's order for four partials: the first lanes of one wavefront).
// What such a call costs is its launches: bucket_clip_flat on 2 K to 16 K elements 7.9 -> 5.3 us a call.
template <int GDT>
__global__ __launch_bounds__(kBlock) void k_clip_one(const Chunk* __restrict__ tab, uint64_t g, uint32_t n, const float* __restrict__ threshold,
                                                      float* norm_out, float* coef_out, int32_t* status) {
  __shared__ double s_w[kWaves];
  __shared__ float s_coef;
  const Entry en = tab != nullptr ? read_entry(tab) : flat_entry(g, n, kFlatChunkNorm, sizeof(typename Grad<GDT>::elem), 0u);
  const float c = *threshold;
  const double ws = sqnorm_chunk<GDT, false, 16>(en);
  if ((threadIdx.x & 63u) == 0) s_w[threadIdx.x >> 6] = ws;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float norm = (float)sqrt((s_w[0] + s_w[2]) + (s_w[1] + s_w[3]));
    int32_t st = 0;
    const float coef = clip_coef(norm, c, st);
    s_coef = coef;
    if (norm_out != nullptr) *norm_out = norm;
    if (coef_out != nullptr) *coef_out = coef;
    if (status != nullptr) *status = st;
  }
  __syncthreads();
  if (s_coef != 1.f) scale_norm_chunk<GDT>(en, s_coef);
}

template <int GDT>
__global__ __launch_bounds__(kBlock) void k_flat_sqnorm(uint64_t g, uint32_t n, double* __restrict__ partials) {
  const Entry en = flat_entry(g, n, kFlatChunkNorm, sizeof(typename Grad<GDT>::elem), blockIdx.x);
  const double ws = sqnorm_chunk<GDT, false, 16>(en);  // cacheable loads: the scale pass reads the bucket again at once
  if ((threadIdx.x & 63u) == 0) partials[(uint64_t)blockIdx.x * kWaves + (threadIdx.x >> 6)] = ws;
}

// Norm, coefficient and status of the bucket from its partial sums (whole workgroup; thread 0 writes the outputs
// if `write_outputs`).  Returns the coefficient to every thread.
__device__ __forceinline__ float flat_coef(const double* __restrict__ partials, uint32_t n_chunks,
                                           const float* __restrict__ threshold, float* norm_out, float* coef_out,
                                           int32_t* status, bool write_outputs, double* s_w, float* s_coef) {
  const double tot = sum_partials(partials, 0, (uint64_t)n_chunks * kWaves, s_w);
  if (threadIdx.x == 0) {
    const float norm = (float)sqrt(tot);
    int32_t st = 0;
    const float coef = clip_coef(norm, *threshold, st);
    *s_coef = coef;
    if (write_outputs) {
      if (norm_out != nullptr) *norm_out = norm;
      if (coef_out != nullptr) *coef_out = coef;
      if (status != nullptr) *status = st;  // written, not ORed
    }
  }
  __syncthreads();
  return *s_coef;
}

// Large buckets only (their partials are too many for every workgroup of the scale launch to add up): one
// workgroup derives the coefficient and leaves it in the scratch header.
__global__ __launch_bounds__(kBlock) void k_flat_finalize(const double* __restrict__ partials, uint32_t n_chunks,
                                                           const float* __restrict__ threshold, float* norm_out,
                                                           float* coef_out, int32_t* status, float* coef_header) {
  __shared__ double s_w[kWaves];
  __shared__ float s_coef;
  const float coef = flat_coef(partials, n_chunks, threshold, norm_out, coef_out, status, true, s_w, &s_coef);
  if (threadIdx.x == 0) *coef_header = coef;
}

// One workgroup per chunk of the squared-norm cut (one workgroup for an empty bucket).  coef_header == nullptr:
// every workgroup derives norm and coefficient from the partial sums itself, as in k_clip_scale, and workgroup 0
// writes the outputs; else the coefficient is read from there.  Then the chunk is scaled.
template <int GDT>
__global__ __launch_bounds__(kBlock) void k_flat_scale(uint64_t g, uint32_t n, uint32_t n_chunks,
                                                        const double* __restrict__ partials,
                                                        const float* __restrict__ threshold, float* norm_out,
                                                        float* coef_out, int32_t* status,
                                                        const float* __restrict__ coef_header) {
  __shared__ double s_w[kWaves];
  __shared__ float s_coef;
  const float coef = coef_header != nullptr
                         ? *coef_header
                         : flat_coef(partials, n_chunks, threshold, norm_out, coef_out, status, blockIdx.x == 0, s_w, &s_coef);
  if (coef == 1.f || blockIdx.x >= n_chunks) return;  // an unclipped bucket is not touched
  scale_norm_chunk<GDT>(flat_entry(g, n, kFlatChunkNorm, sizeof(typename Grad<GDT>::elem), blockIdx.x), coef);
}

// Plain device-to-device copy (16-byte pieces, then single bytes).  It exists so
// that hardware counters can be calibrated against a kernel whose HBM traffic is
// known exactly: nbytes read, nbytes written.
__global__ __launch_bounds__(kBlock) void k_copy(uint8_t* __restrict__ dst, const uint8_t* __restrict__ src,
                                                  uint64_t nbytes) {
  const uint64_t nvec = nbytes / 16u;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < nvec; i += stride)
    reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(src)[i];
  for (uint64_t i = nvec * 16u + (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < nbytes; i += stride) dst[i] = src[i];
}

// Compile-time variants are picked from run-time switches through these helpers.
template <typename F>
void pick2(bool a, bool b, F f) {
  if (a) {
    if (b) f(std::true_type{}, std::true_type{});
    else f(std::true_type{}, std::false_type{});
  } else {
    if (b) f(std::false_type{}, std::true_type{});
    else f(std::false_type{}, std::false_type{});
  }
}
template <typename F>
void pick_gdt(int gdt, F f) {
  if (gdt == BCA_GRAD_F32) f(std::integral_constant<int, BCA_GRAD_F32>{});
  else if (gdt == BCA_GRAD_F16) f(std::integral_constant<int, BCA_GRAD_F16>{});
  else f(std::integral_constant<int, BCA_GRAD_BF16>{});
}
template <typename F>
void pick_unroll(uint32_t u, F f) {
  if (u == 1) f(std::integral_constant<uint32_t, 1>{});
  else if (u == 2) f(std::integral_constant<uint32_t, 2>{});
  else f(std::integral_constant<uint32_t, 4>{});
}

}  // namespace

// ---- launchers --------------------------------------------------------------------

hipError_t launch_sqnorm(int gdt, const Chunk* table, uint32_t c0, uint32_t n, double* partials, int32_t* status,
                         const Launch& L, hipStream_t stream) {
  if (n == 0 && status == nullptr) return hipSuccess;  // with a status word the launch still has to clear it
  pick2(!L.g_keep, L.staged, [&](auto nt, auto st) {
    constexpr bool NT = decltype(nt)::value, ST = decltype(st)::value;
    pick_gdt(gdt, [&](auto gd) {
      constexpr int GDT = decltype(gd)::value;
      // a launch that does not fill the GPU (one bucket) keeps a whole 16 Ki chunk in flight per workgroup
      if (L.grid <= kSmallNormGrid)
        hipLaunchKernelGGL((k_sqnorm<GDT, NT, ST, 16>), dim3(L.grid), dim3(kBlock), 0, stream, table, c0, n, partials,
                           status);
      else
        hipLaunchKernelGGL((k_sqnorm<GDT, NT, ST, 8>), dim3(L.grid), dim3(kBlock), 0, stream, table, c0, n, partials,
                           status);
    });
  });
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, uint64_t nbytes, hipStream_t stream) {
  if (nbytes == 0) return hipSuccess;
  const uint64_t want = (nbytes / 16u + kBlock - 1) / kBlock;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(want, 1), 1u << 20);
  hipLaunchKernelGGL(k_copy, dim3(grid), dim3(kBlock), 0, stream, (uint8_t*)dst, (const uint8_t*)src, nbytes);
  return hipGetLastError();
}

hipError_t launch_clip_scale(int gdt, const Chunk* norm_tab, uint32_t cn0, uint32_t n, const uint32_t* bucket_chunk_off,
                             uint32_t b0, uint32_t b1, const double* partials, const float* thresholds, float* norms,
                             float* coefs, int32_t* status, hipStream_t stream) {
  pick_gdt(gdt, [&](auto gd) {
    hipLaunchKernelGGL((k_clip_scale<decltype(gd)::value>), dim3(std::max(n, 1u)), dim3(kBlock), 0, stream, norm_tab, cn0, n,
                       bucket_chunk_off, b0, b1, partials, thresholds, norms, coefs, status);
  });
  return hipGetLastError();
}

hipError_t launch_step(int gdt, const StepState& st, const uint32_t* work, uint32_t n_work, const float* thresholds,
                       float* norms, float* coefs, int32_t* status, bool write_back, const AdamK& k, uint32_t unroll,
                       bool tickets, bool lamb, hipEvent_t between, hipStream_t stream) {
  // Plans of few items finish themselves (kSelfFinishItems); with events to be recorded in between there are two launches.
  const bool plain = !lamb && !tickets && unroll == 1;
  const bool self = plain && between == nullptr && n_work <= kSelfFinishItems;
  if (n_work != 0) {
    if (self) {
      pick_gdt(gdt, [&](auto gd) {
        constexpr int GDT = decltype(gd)::value;
        if (write_back)
          hipLaunchKernelGGL((k_step<GDT, true, 1, false, false, true>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                             thresholds, norms, coefs, k, status);
        else
          hipLaunchKernelGGL((k_step<GDT, false, 1, false, false, true>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                             thresholds, norms, coefs, k, status);
      });
      return hipGetLastError();
    }
    if (plain && n_work <= kEarlyItems) {
      pick_gdt(gdt, [&](auto gd) {
        constexpr int GDT = decltype(gd)::value;
        if (write_back)
          hipLaunchKernelGGL((k_step<GDT, true, 1, false, false, false, true>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                             thresholds, norms, coefs, k, status);
        else
          hipLaunchKernelGGL((k_step<GDT, false, 1, false, false, false, true>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                             thresholds, norms, coefs, k, status);
      });
    } else if (lamb) {  // one variant per gradient type and write-back setting: items by workgroup index, no unrolling
      pick_gdt(gdt, [&](auto gd) {
        constexpr int GDT = decltype(gd)::value;
        if (write_back)
          hipLaunchKernelGGL((k_step<GDT, true, 1, false, true>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                             thresholds, norms, coefs, k, status);
        else
          hipLaunchKernelGGL((k_step<GDT, false, 1, false, true>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                             thresholds, norms, coefs, k, status);
      });
    } else {
      pick_unroll(unroll, [&](auto uu) {
        constexpr uint32_t U = decltype(uu)::value;
        pick2(tickets, write_back, [&](auto tk, auto wb) {
          constexpr bool TK = decltype(tk)::value, WB = decltype(wb)::value;
          pick_gdt(gdt, [&](auto gd) {
            constexpr int GDT = decltype(gd)::value;
            hipLaunchKernelGGL((k_step<GDT, WB, U, TK, false>), dim3(n_work), dim3(kBlock), 0, stream, st, work, n_work,
                               thresholds, norms, coefs, k, status);
          });
        });
      });
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (between != nullptr) (void)hipEventRecord(between, stream);
  // the finish kernel: skipped items (same arithmetic whatever the unrolling, so one variant), status, next epoch
  pick2(lamb, write_back, [&](auto lm, auto wb) {
    constexpr bool LM = decltype(lm)::value, WB = decltype(wb)::value;
    pick_gdt(gdt, [&](auto gd) {
      constexpr int GDT = decltype(gd)::value;
      hipLaunchKernelGGL((k_finish<GDT, WB, 1, LM ? kModeLamb : kModeAdam>), dim3(1), dim3(kBlock), 0, stream, st, status,
                         k);
    });
  });
  return hipGetLastError();
}

hipError_t launch_finalize(const double* partials, const uint32_t* bucket_chunk_off, uint32_t b0, uint32_t b1,
                           const float* thresholds, float* norms, float* coefs, int32_t* status, double* bucket_sq,
                           hipStream_t stream) {
  if (b1 <= b0) return hipSuccess;
  hipLaunchKernelGGL(k_finalize, dim3(b1 - b0), dim3(kBlock), 0, stream, partials, bucket_chunk_off, b0, thresholds,
                     norms, coefs, status, bucket_sq);
  return hipGetLastError();
}

hipError_t launch_norms(int gdt, const StepState& st, uint32_t n, uint32_t n_buckets, uint32_t n_filled, bool whole, const float* thresholds,
                        float* norms, float* coefs, double* bucket_sq, int32_t* status, hipStream_t stream) {
  pick_gdt(gdt, [&](auto gd) {
    hipLaunchKernelGGL((k_norms<decltype(gd)::value>), dim3(std::max(n, 1u)), dim3(kBlock), 0, stream, st, n, n_buckets, n_filled, whole,
                       thresholds, norms, coefs, bucket_sq, status);
  });
  return hipGetLastError();
}

hipError_t launch_whole_coef(const double* bucket_sq, uint32_t n_buckets, const float* c, float* whole_norm,
                             float* coefs, int32_t* status, hipStream_t stream) {
  hipLaunchKernelGGL(k_whole_coef, dim3(1), dim3(kBlock), 0, stream, bucket_sq, n_buckets, c, whole_norm, coefs,
                     status);
  return hipGetLastError();
}

hipError_t launch_coefs(uint32_t b0, uint32_t b1, const float* thresholds, const float* norms, float* coefs,
                        int32_t* status, hipStream_t stream) {
  hipLaunchKernelGGL(k_coefs, dim3(1), dim3(kBlock), 0, stream, b0, b1, thresholds, norms, coefs, status);
  return hipGetLastError();
}

hipError_t launch_scale(int gdt, const Chunk* table, uint32_t c0, uint32_t n, const float* coefs, const Launch& L,
                        hipStream_t stream) {
  if (n == 0) return hipSuccess;
  // The scaled gradients are about to be read again (by the all-reduce or by Adam): plain stores.
  pick_unroll(L.unroll, [&](auto uu) {
    constexpr uint32_t U = decltype(uu)::value;
    pick_gdt(gdt, [&](auto gd) {
      constexpr int GDT = decltype(gd)::value;
      if (L.staged)
        hipLaunchKernelGGL((k_scale<GDT, U, false, true>), dim3(L.grid), dim3(kBlock), 0, stream, table, c0, n, coefs);
      else
        hipLaunchKernelGGL((k_scale<GDT, U, false, false>), dim3(L.grid), dim3(kBlock), 0, stream, table, c0, n, coefs);
    });
  });
  return hipGetLastError();
}

template <int GDT, uint32_t U, bool GNT, bool ST>
static void launch_adam_t(const Chunk* table, uint32_t c0, uint32_t n, const float* coefs, bool write_back,
                          const int32_t* skip_status, const AdamK& k, const Launch& L, hipStream_t stream) {
  if (coefs == nullptr)
    hipLaunchKernelGGL((k_adam<GDT, false, false, U, GNT, ST>), dim3(L.grid), dim3(kBlock), L.lds, stream, table, c0, n,
                       coefs, skip_status, k, L.order);
  else if (!write_back)
    hipLaunchKernelGGL((k_adam<GDT, true, false, U, GNT, ST>), dim3(L.grid), dim3(kBlock), L.lds, stream, table, c0, n,
                       coefs, skip_status, k, L.order);
  else
    hipLaunchKernelGGL((k_adam<GDT, true, true, U, GNT, ST>), dim3(L.grid), dim3(kBlock), L.lds, stream, table, c0, n,
                       coefs, skip_status, k, L.order);
}

hipError_t launch_adam(int gdt, const Chunk* table, uint32_t c0, uint32_t n, const float* coefs, bool write_back,
                       const int32_t* skip_status, const AdamK& k, const Launch& L, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  pick_unroll(L.unroll, [&](auto uu) {
    constexpr uint32_t U = decltype(uu)::value;
    pick2(!L.g_keep, L.staged, [&](auto gnt, auto st) {
      constexpr bool GNT = decltype(gnt)::value, ST = decltype(st)::value;
      pick_gdt(gdt, [&](auto gd) {
        launch_adam_t<decltype(gd)::value, U, GNT, ST>(table, c0, n, coefs, write_back, skip_status, k, L, stream);
      });
    });
  });
  return hipGetLastError();
}

hipError_t launch_lamb_moments(int gdt, const Chunk* table, uint32_t n, const float* coefs, bool write_back,
                               double* sums, bool keep, const AdamK& k, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  pick2(keep, write_back, [&](auto kp, auto wbk) {
    constexpr bool KEEP = decltype(kp)::value, WB = decltype(wbk)::value;
    pick_gdt(gdt, [&](auto gd) {
      constexpr int GDT = decltype(gd)::value;
      if (coefs == nullptr)
        hipLaunchKernelGGL((k_lamb_moments<GDT, false, false, KEEP>), dim3(n), dim3(kBlock), 0, stream, table, n, coefs, sums, k);
      else
        hipLaunchKernelGGL((k_lamb_moments<GDT, true, WB, KEEP>), dim3(n), dim3(kBlock), 0, stream, table, n, coefs, sums, k);
    });
  });
  return hipGetLastError();
}

hipError_t launch_lamb(int gdt, const StepState& st, const LambState& ls, const uint32_t* work, uint32_t n_work, bool clip,
                       const float* thresholds, float* norms, float* coefs, int32_t* status, bool write_back, const AdamK& k,
                       hipStream_t stream) {
  hipError_t e = hipSuccess;
  pick_gdt(gdt, [&](auto gd) {
    constexpr int GDT = decltype(gd)::value;
    if (n_work != 0) {
      if (!clip)
        hipLaunchKernelGGL((k_lamb<GDT, false, false>), dim3(n_work), dim3(kBlock), 0, stream, st, ls, work, thresholds, norms, coefs, k);
      else if (write_back)
        hipLaunchKernelGGL((k_lamb<GDT, true, true>), dim3(n_work), dim3(kBlock), 0, stream, st, ls, work, thresholds, norms, coefs, k);
      else
        hipLaunchKernelGGL((k_lamb<GDT, true, false>), dim3(n_work), dim3(kBlock), 0, stream, st, ls, work, thresholds, norms, coefs, k);
      e = hipGetLastError();
    }
    if (e != hipSuccess || !clip) return;
    if (write_back) hipLaunchKernelGGL((k_lamb_late<GDT, true>), dim3(kLambLateWorkers), dim3(kBlock), 0, stream, st, ls, k);
    else hipLaunchKernelGGL((k_lamb_late<GDT, false>), dim3(kLambLateWorkers), dim3(kBlock), 0, stream, st, ls, k);
    e = hipGetLastError();
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lamb_tail, dim3(std::max((ls.first_end - ls.first_large) * kLambItemChunks, kLambTailWorkers)), dim3(kBlock), 0, stream, st, ls, status, k);
  return hipGetLastError();
}

hipError_t launch_hyper(const bca_adam_device* dev, AdamK* out, hipStream_t stream) {
  hipLaunchKernelGGL(k_hyper, dim3(1), dim3(64), 0, stream, dev, out);
  return hipGetLastError();
}

hipError_t launch_lamb_trust(const double* sums, const uint32_t* tensor_off, uint32_t n_tensors, const AdamK& k,
                             float* trust, float* scale, hipStream_t stream) {
  if (n_tensors == 0) return hipSuccess;
  hipLaunchKernelGGL(k_lamb_trust, dim3(n_tensors), dim3(kTrustBlock), 0, stream, sums, tensor_off, k, trust, scale);
  return hipGetLastError();
}

hipError_t launch_clip_one(int gdt, const Chunk* tab, uint64_t g, uint32_t n, const float* threshold, float* norm, float* coef, int32_t* status,
                           hipStream_t stream) {
  pick_gdt(gdt, [&](auto gd) {
    hipLaunchKernelGGL((k_clip_one<decltype(gd)::value>), dim3(1), dim3(kBlock), 0, stream, tab, g, n, threshold, norm, coef, status);
  });
  return hipGetLastError();
}

// Device address of `scratch` on each device, looked up once per device with that device current
// (every device holds its own copy of the array at its own address).  Host code never uses the
// array's name for anything else: as an expression it is a host-side stand-in, not a device address.
static void* g_flat_scratch[kFlatMaxDevices];
static hipError_t g_flat_scratch_err[kFlatMaxDevices];
static std::once_flag g_flat_scratch_once[kFlatMaxDevices];

hipError_t launch_clip_flat(int device, int gdt, void* g, uint64_t n, const float* threshold, float* norm, float* coef,
                            int32_t* status, hipStream_t stream) {
  std::call_once(g_flat_scratch_once[device], [device] {
    void* ptr = nullptr;
    g_flat_scratch_err[device] = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_flat_scratch[device] = g_flat_scratch_err[device] == hipSuccess ? ptr : nullptr;
  });
  if (g_flat_scratch_err[device] != hipSuccess) return g_flat_scratch_err[device];
  unsigned char* base = static_cast<unsigned char*>(g_flat_scratch[device]);
  if (base == nullptr) return hipErrorInvalidSymbol;
  float* coef_header = reinterpret_cast<float*>(base);
  double* partials = reinterpret_cast<double*>(base + kFlatHeaderBytes);
  const uint32_t n_norm = (uint32_t)((n + kFlatChunkNorm - 1) / kFlatChunkNorm);
  const uint64_t ga = (uint64_t)(uintptr_t)g;
  const bool large = n_norm > kMaxChunksForInlineFinalize;
  hipError_t e = hipSuccess;
  if (n_norm == 1) return launch_clip_one(gdt, nullptr, ga, (uint32_t)n, threshold, norm, coef, status, stream);
  // Nothing in the scratch array has to start at zero: every partial (and the header) that a later kernel of the
  // call reads is written by an earlier kernel of this same call.
  if (n_norm != 0) {
    pick_gdt(gdt, [&](auto gd) {
      hipLaunchKernelGGL((k_flat_sqnorm<decltype(gd)::value>), dim3(n_norm), dim3(kBlock), 0, stream, ga, (uint32_t)n, partials);
    });
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (large) {
    hipLaunchKernelGGL(k_flat_finalize, dim3(1), dim3(kBlock), 0, stream, partials, n_norm, threshold, norm, coef, status,
                       coef_header);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  pick_gdt(gdt, [&](auto gd) {
    hipLaunchKernelGGL((k_flat_scale<decltype(gd)::value>), dim3(std::max(n_norm, 1u)), dim3(kBlock), 0, stream, ga, (uint32_t)n, n_norm,
                       partials, threshold, norm, coef, status, large ? coef_header : nullptr);
  });
  return hipGetLastError();
}

hipError_t launch_lamb_update(const Chunk* table, uint32_t n, const float* scale, const AdamK& k, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_lamb_update, dim3(n), dim3(kBlock), 0, stream, table, n, scale, k);
  return hipGetLastError();
}

}  // namespace bca
