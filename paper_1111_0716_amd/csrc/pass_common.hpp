// Device helpers shared by the register-line passes (pass_reg.hip) and the
// line passes of general grids (pass_line.hip).
#pragma once

#include "fft_lds.hpp"

namespace fock {

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
  const double b = 2.0 * nP + 1.0;
  int r = static_cast<int>((b - sqrt(b * b - 8.0 * pi)) * 0.5);
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
  return reinterpret_cast<C*>(reinterpret_cast<uintptr_t>(u) + o);
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
