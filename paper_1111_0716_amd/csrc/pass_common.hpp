// Device helpers of the three-pass kernels (pass_line.hip, plane_fft.hpp,
// pass_reg.hip, energy_lds.hip), the register-line DFT (dft_reg.hip) and the
// reductions (kernels.hip).
#pragma once

#include <type_traits>

#include "fft_lds.hpp"

namespace fock {

// ---------------------------------------------------------------------------
// deterministic block reduction of a double (kBlock threads, wave64)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) {
    for (int w = 0; w < kBlock / 64; ++w) t += red[w];
  }
  __syncthreads();
  return t;  // valid in thread 0
}

// one step of a compensated (Neumaier) sum
__device__ __forceinline__ void neumaier(double& sum, double& comp, double x) {
  const double t = sum + x;
  comp += (fabs(sum) >= fabs(x)) ? (sum - t) + x : (x - t) + sum;
  sum = t;
}

// Loads issued in batches with the next batch in flight while the current one
// is consumed: only two batches of operands are live beside the line, and a
// phase costs (elements / batch) - 1 memory latencies at most.
constexpr int kRegB = 8;

// Compiler-only barrier: loads are not hoisted across it.
__device__ __forceinline__ void reg_fence() { asm volatile("" ::: "memory"); }

// the largest batch size <= want that divides L
__host__ __device__ constexpr int batch_of(int L, int want) {
  int b = want < L ? want : L;
  while (L % b != 0) --b;
  return b;
}

// Output and partner slots (o, p) of pair slot pi of an apply batch: pi =
// o nP + p, or for a block paired with itself (tri) the unordered pairs
// o <= p, row-major over the upper triangle (row o starts at tri_slot(o, o)).
__host__ __device__ constexpr size_t tri_slot(int o, int p, int n) {
  return static_cast<size_t>(o) * n - static_cast<size_t>(o) * (o - 1) / 2 + static_cast<size_t>(p - o);
}

__device__ __forceinline__ void batch_pair(int pi, int nP, int tri, int* o, int* p) {
  if (!tri) {
    *o = pi / nP;
    *p = pi - *o * nP;
    return;
  }
  // FP32 estimate of the row (the block index is uniform: one scalar value),
  // then exact
  const float b = 2.0f * nP + 1.0f;
  int r = static_cast<int>((b - __builtin_amdgcn_sqrtf(fmaxf(b * b - 8.0f * pi, 0.0f))) * 0.5f);
  r = __builtin_amdgcn_readfirstlane(r);
  r = r < 0 ? 0 : (r > nP - 1 ? nP - 1 : r);
  while (r > 0 && tri_slot(r, r, nP) > static_cast<size_t>(pi)) --r;
  while (r + 1 < nP && tri_slot(r + 1, r + 1, nP) <= static_cast<size_t>(pi)) ++r;
  *o = r;
  *p = r + static_cast<int>(static_cast<size_t>(pi) - tri_slot(r, r, nP));
}

// complex value in another precision
template <typename C, typename CI>
__device__ __forceinline__ C cvt(CI v) {
  using T = decltype(C{}.x);
  return C{static_cast<T>(v.x), static_cast<T>(v.y)};
}

// Pencil lines with the line count known only at run time: the address of
// element j is a wave-uniform base (scalar registers) plus the lane's 32-bit
// byte offset, so the loads of a line take no 64-bit address per element.
template <typename C>
__device__ __forceinline__ C* lane_at(C* u, unsigned o) {
  using Byte = typename std::conditional<std::is_const<C>::value, const char, char>::type;
  return reinterpret_cast<C*>(reinterpret_cast<Byte*>(u) + o);
}

// STREAM: a pair buffer larger than the caches goes through memory once per pass,
// and its accesses are marked non-temporal, so that they do not push the
// orbitals and tables out of L2 (the accumulate's reads included, although a
// pair is read once for each of its orders: the two reads are far apart).  32^3
// 4x4x4 k FP32 step 367.5 -> 336.6 ms (stores alone 344.9, all but the
// accumulate's reads 340.9), 64^3 Gamma FP32 17.85 -> 17.05; 72^3 FP32 77.0 ->
// 76.5.  A buffer that the caches hold is read by the next pass from there, and
// marked accesses lose that: pair_streams (fock_internal.hpp) has the line.
template <bool STREAM, typename C>
__device__ __forceinline__ C stream_load(const C* p) {
  typedef decltype(C{}.x) V2 __attribute__((ext_vector_type(2)));
  if constexpr (!STREAM) return *p;
  const V2 v = __builtin_nontemporal_load(reinterpret_cast<const V2*>(p));
  return C{v.x, v.y};
}
template <bool STREAM, typename C>
__device__ __forceinline__ void stream_store(C* p, C a) {
  typedef decltype(C{}.x) V2 __attribute__((ext_vector_type(2)));
  if constexpr (!STREAM) {
    *p = a;
    return;
  }
  V2 v;
  v.x = a.x;
  v.y = a.y;
  __builtin_nontemporal_store(v, reinterpret_cast<V2*>(p));
}
// Loads and stores at a wave-uniform base plus the lane's 32-bit byte offset
// (lane_at's addresses): the base goes through an empty asm in scalar
// registers, so that it is formed there, and the access takes the two as they
// are instead of one 64-bit vector addition for every element.
template <typename V>
__device__ __forceinline__ __attribute__((address_space(1))) V* lane_ptr(const void* u, unsigned o) {
  typedef __attribute__((address_space(1))) char* Bytes;
  Bytes b = (Bytes)(const_cast<void*>(u));
  asm("" : "+s"(b));
  return (__attribute__((address_space(1))) V*)(b + o);
}
template <typename R> struct lane_vec { typedef decltype(R{}.x) type __attribute__((ext_vector_type(2))); };
template <> struct lane_vec<float> { typedef float type; };
template <> struct lane_vec<double> { typedef double type; };
template <typename R, typename V>
__device__ __forceinline__ R from_vec(V v) {
  if constexpr (sizeof(R) == sizeof(v) && std::is_arithmetic<R>::value)
    return v;
  else
    return R{v.x, v.y};
}
template <bool STREAM = false, typename C>
__device__ __forceinline__ C lane_load(const C* u, unsigned o) {
  const auto* p = lane_ptr<typename lane_vec<C>::type>(u, o);
  if constexpr (STREAM) return from_vec<C>(__builtin_nontemporal_load(p));
  return from_vec<C>(*p);
}
template <bool STREAM = false, typename C>
__device__ __forceinline__ void lane_store(C* u, unsigned o, C a) {
  typename lane_vec<C>::type v = {a.x, a.y};
  auto* p = lane_ptr<typename lane_vec<C>::type>(u, o);
  if constexpr (STREAM)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// v, through an empty asm the compiler cannot see through: addresses built
// from the copy are formed where they are used instead of being kept live
// (two registers each) across the transform in between
__device__ __forceinline__ unsigned opaque(unsigned v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Batch pairs are pi = o nP + p (output o0 + o, partner parts[p]).  One
// launch serves the batch's outputs (blockIdx.y = o < nO) and, for a batch of
// unordered pairs of two blocks (mirror), also its partners (blockIdx.y =
// nO + p): the outputs are disjoint, so the two halves never write the same
// band.
//   output o:    W of pair (o, p) for every p, times u_p.
//   partner p:   the partner is the output; for every o the pair's W_{o p}
//                gives W_{p o} = conj(W_{o p}), times u_{o0+o}.
//   tri (a block paired with itself, unordered pairs o <= p at tri_slot):
//                 output o takes W_{o p} from slot (o, p) for p >= o and
//                 conj(W_{p o}) from slot (p, o) for p < o.
// The global band index of the orbital that multiplies W, the pair slot, and
// whether the slot holds the conjugate of the W wanted.
__device__ __forceinline__ void acc_source(bool mirror, int j, int blk, int o0, int nP, int tri, int nbands,
                                           const int2* __restrict__ parts, int* band, size_t* pair, bool* cj) {
  if (mirror) {
    *band = o0 + j;
    *pair = static_cast<size_t>(j) * nP + blk;
    *cj = true;
  } else {
    const int2 r = parts[j];
    *band = r.x * nbands + r.y;
    if (tri) {
      *pair = j >= blk ? tri_slot(blk, j, nP) : tri_slot(j, blk, nP);
      *cj = j < blk;
    } else {
      *pair = static_cast<size_t>(blk) * nP + j;
      *cj = false;
    }
  }
}

}  // namespace fock
