// In-LDS FFT of a plane (or a stack of planes) with lengths known at run
// time, in two radix passes per axis.
//
// A length n = a b (a, b <= 10, a = 1 for the lengths of one pass) is
// transformed by decimation in frequency in place:
//
//   pass a   for every j < b: the a samples j + r b, DFT_a, times W_n^{j r},
//            back to the same places
//   pass b   for every r < a: the b values r b + j, DFT_b, back to the same
//            places: position r b + k holds the frequency r + a k
//
// The inverse runs the passes backwards (conjugate twiddles before DFT_a), so
// a spectrum that is only multiplied point by point never has to be sorted:
// the kernel table is stored in the order of the positions instead.  Every
// butterfly writes where it read, so a pass needs one barrier, not two, and
// the radices are the only compile-time parameters.
#pragma once

#include "fft_lds.hpp"
#include "fock_internal.hpp"

namespace fock {

template <int S, typename C> struct Dft<6, S, C> {  // 2 x 3, prime factors: no twiddles
  static __device__ __forceinline__ void run(C* x) {
    C e[3] = {x[0], x[2], x[4]}, o[3] = {x[3], x[5], x[1]};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const C a = e[i], b = o[i];
      e[i] = cadd(a, b);
      o[i] = csub(a, b);
    }
    Dft<3, S, C>::run(e);
    Dft<3, S, C>::run(o);
    x[0] = e[0];
    x[4] = e[1];
    x[2] = e[2];
    x[3] = o[0];
    x[1] = o[1];
    x[5] = o[2];
  }
};

template <int S, typename C> struct Dft<9, S, C> {  // 3 x 3
  static __device__ __forceinline__ void run(C* x) {
    using T = decltype(x[0].x);
    // e^{S 2 pi i k / 9}, k = 1, 2, 4
    const C w1 = C{T(0.7660444431189780352023926505554167), S * T(0.6427876096865393263226434099072632)};
    const C w2 = C{T(0.1736481776669303488517166267693148), S * T(0.9848077530122080593667430245895230)};
    const C w4 = C{T(-0.9396926207859083840541092773247315), S * T(0.3420201433256687330440996146822596)};
    C a[3] = {x[0], x[3], x[6]}, b[3] = {x[1], x[4], x[7]}, c[3] = {x[2], x[5], x[8]};
    Dft<3, S, C>::run(a);
    Dft<3, S, C>::run(b);
    Dft<3, S, C>::run(c);
    b[1] = cmul(b[1], w1);
    b[2] = cmul(b[2], w2);
    c[1] = cmul(c[1], w2);
    c[2] = cmul(c[2], w4);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      C v[3] = {a[k], b[k], c[k]};
      Dft<3, S, C>::run(v);
      x[k] = v[0];
      x[k + 3] = v[1];
      x[k + 6] = v[2];
    }
  }
};

template <int S, typename C> struct Dft<10, S, C> {  // 2 x 5, prime factors: no twiddles
  static __device__ __forceinline__ void run(C* x) {
    C e[5] = {x[0], x[2], x[4], x[6], x[8]}, o[5] = {x[5], x[7], x[9], x[1], x[3]};
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const C a = e[i], b = o[i];
      e[i] = cadd(a, b);
      o[i] = csub(a, b);
    }
    Dft<5, S, C>::run(e);
    Dft<5, S, C>::run(o);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      x[(6 * k) % 10] = e[k];
      x[(5 + 6 * k) % 10] = o[k];
    }
  }
};

// `call` with the compile-time radix R
#define FOCK_RADIX(r, call)                            \
  switch (r) {                                         \
    case 2: { constexpr int R = 2; call; break; }      \
    case 3: { constexpr int R = 3; call; break; }      \
    case 4: { constexpr int R = 4; call; break; }      \
    case 5: { constexpr int R = 5; call; break; }      \
    case 6: { constexpr int R = 6; call; break; }      \
    case 8: { constexpr int R = 8; call; break; }      \
    case 9: { constexpr int R = 9; call; break; }      \
    default: { constexpr int R = 10; call; break; }    \
  }

template <typename C>
__device__ __forceinline__ C cconj(C a) { return C{a.x, -a.y}; }

// W^t of the table for S = -1, its conjugate for S = +1
template <int S, typename C>
__device__ __forceinline__ C twid(C w) { return S < 0 ? w : cconj(w); }

// axis 2, pass a (or the only pass), from the planes in memory: consecutive
// lanes take consecutive elements, so every load is coalesced
template <int R, int S, typename C>
__device__ __forceinline__ void ax2_load(C* s, const C* __restrict__ src, const PlaneGeo& g, int gc,
                                         const C* __restrict__ tw) {
  const int M = g.n2 / R, mn = M * g.n3, total = gc * mn;
  const float rmn = 1.0f / static_cast<float>(mn), r3 = 1.0f / static_cast<float>(g.n3);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int gg = fdiv(idx, rmn), rem = idx - gg * mn;
    const int m = fdiv(rem, r3), j3 = rem - m * g.n3;
    const C* p = src + (gg * (g.n2 * g.n3) + rem);
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = p[r * mn];
    Dft<R, S, C>::run(v);
    C* d = s + (gg * g.n2 + m) * g.pitch + j3;
    d[0] = v[0];
#pragma unroll
    for (int r = 1; r < R; ++r) d[r * M * g.pitch] = M > 1 ? cmul(v[r], twid<S>(tw[r * m])) : v[r];
  }
}

// axis 2, inverse pass a, to the planes in memory
template <int R, int S, typename C>
__device__ __forceinline__ void ax2_store(const C* s, C* __restrict__ dst, const PlaneGeo& g, int gc, const C* tw) {
  const int M = g.n2 / R, mn = M * g.n3, total = gc * mn;
  const float rmn = 1.0f / static_cast<float>(mn), r3 = 1.0f / static_cast<float>(g.n3);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int gg = fdiv(idx, rmn), rem = idx - gg * mn;
    const int m = fdiv(rem, r3), j3 = rem - m * g.n3;
    const C* p = s + (gg * g.n2 + m) * g.pitch + j3;
    C v[R];
    v[0] = p[0];
#pragma unroll
    for (int r = 1; r < R; ++r) {
      v[r] = p[r * M * g.pitch];
      if (M > 1) v[r] = cmul(v[r], twid<S>(tw[r * m]));
    }
    Dft<R, S, C>::run(v);
    C* d = dst + (gg * (g.n2 * g.n3) + rem);
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * mn] = v[r];
  }
}

// axis 2, pass b
template <int R, int S, typename C>
__device__ __forceinline__ void ax2_b(C* s, const PlaneGeo& g, int gc) {
  const int total = gc * g.a2 * g.n3;
  const float r3 = 1.0f / static_cast<float>(g.n3);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int gk = fdiv(idx, r3), j3 = idx - gk * g.n3;
    C* p = s + gk * R * g.pitch + j3;
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = p[r * g.pitch];
    Dft<R, S, C>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) p[r * g.pitch] = v[r];
  }
}

// axis 3: consecutive lanes take consecutive rows, whose pitch is odd, so the
// lanes spread over all LDS banks
// pass a (S = -1: forward, twiddles after; INV: backwards, twiddles before)
template <int R, int S, bool INV, typename C>
__device__ __forceinline__ void ax3_a(C* s, const PlaneGeo& g, int rows, const C* tw) {
  const int total = rows * g.b3;
  const float rr = 1.0f / static_cast<float>(rows);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int j = fdiv(idx, rr), row = idx - j * rows;
    C* p = s + row * g.pitch + j;
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[r] = p[r * g.b3];
      if (INV && r > 0) v[r] = cmul(v[r], twid<S>(tw[r * j]));
    }
    Dft<R, S, C>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) p[r * g.b3] = !INV && r > 0 ? cmul(v[r], twid<S>(tw[r * j])) : v[r];
  }
}

// axis 3, pass b (or the only pass)
template <int R, int S, typename C>
__device__ __forceinline__ void ax3_b(C* s, const PlaneGeo& g, int rows) {
  const int total = rows * g.a3;
  const float rr = 1.0f / static_cast<float>(rows);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int k1 = fdiv(idx, rr), row = idx - k1 * rows;
    C* p = s + row * g.pitch + k1 * R;
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = p[r];
    Dft<R, S, C>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = v[r];
  }
}

// axis 3, pass b, times the kernel and back (BACK), with the energy sum (EN).
// v: the tile's kernel values in the order [k2][k1][row]
template <int R, bool EN, bool BACK, typename C, typename T>
__device__ __forceinline__ void ax3_kernel(C* s, const PlaneGeo& g, int rows, const T* __restrict__ v, double* en) {
  const int total = rows * g.a3;
  const float rr = 1.0f / static_cast<float>(rows);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int k1 = fdiv(idx, rr), row = idx - k1 * rows;
    T vv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) vv[r] = v[r * total + idx];
    C* p = s + row * g.pitch + k1 * R;
    C x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = p[r];
    Dft<R, -1, C>::run(x);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if constexpr (EN) {
        const double px = static_cast<double>(x[r].x), py = static_cast<double>(x[r].y);
        *en += static_cast<double>(vv[r]) * (px * px + py * py);
      }
      if constexpr (BACK) x[r] = cscale(x[r], vv[r]);
    }
    if constexpr (BACK) {
      Dft<R, +1, C>::run(x);
#pragma unroll
      for (int r = 0; r < R; ++r) p[r] = x[r];
    }
  }
}

}  // namespace fock
