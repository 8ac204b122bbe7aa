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
#include "pass_common.hpp"

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

// n = a b with both at most 10 (never 7), the least a + b; a = 1 if n itself is one radix
__host__ __device__ constexpr int radix_a(int n) {
  if (n <= 10) return 1;
  int a = 1, best = 1000;
  for (int x = 2; x <= 10; ++x) {
    if (n % x != 0 || x == 7 || n / x > 10 || n / x < x) continue;
    if (x + n / x < best) {
      best = x + n / x;
      a = x;
    }
  }
  return a;
}

// every {2,3,5}-smooth axis length
#define FOCK_SMOOTH_L(X)                                                                                       \
  X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12) X(15) X(16) X(18) X(20) X(24) X(25) X(27) X(30) X(32) X(36) \
  X(40) X(45) X(48) X(50) X(54) X(60) X(64) X(72)

// 1 / n to one unit in the last place: fdiv's quotients stay exact (its error
// is then at most 5 2^-24 idx/n, under 0.32/n at idx < 2^20)
__device__ __forceinline__ float rcp_of(int n) { return __builtin_amdgcn_rcpf(static_cast<float>(n)); }

template <typename C>
__device__ __forceinline__ C cconj(C a) { return C{a.x, -a.y}; }

// W^t of the table for S = -1, its conjugate for S = +1
template <int S, typename C>
__device__ __forceinline__ C twid(C w) { return S < 0 ? w : cconj(w); }

// Twiddles of a length n = a b: W_n^{r j} at (r - 1) b + j, 1 <= r < a, j < b
// (plan.cpp), at twiddle_offset(n) of the plan's table.
constexpr int twiddle_count(int n) { return (radix_a(n) - 1) * (n / radix_a(n)); }

// axis 2, pass a (or the only pass), from the planes in memory: consecutive lanes take consecutive elements, so every load is
// coalesced
template <int N, int S, bool STREAM, typename C>
__device__ __forceinline__ void ax2_load(C* s, const C* src, int n3, int pitch, int gc,
                                         const C* __restrict__ tw) {
  constexpr int A = radix_a(N), R = A > 1 ? A : N, M = N / R;
  const int mn = M * n3, total = gc * mn;
  const float rmn = rcp_of(mn), r3 = rcp_of(n3);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int gg = gc > 1 ? fdiv(idx, rmn) : 0, rem = idx - __mul24(gg, mn);
    const int m = M > 1 ? fdiv(rem, r3) : 0, j3 = rem - __mul24(m, n3);
    const unsigned o = static_cast<unsigned>(__mul24(gg, N * n3) + rem) * sizeof(C);
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = stream_load<STREAM>(lane_at(src + r * mn, o));
    Dft<R, S, C>::run(v);
    if constexpr (M > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = cmul(v[r], twid<S>(tw[(r - 1) * M + m]));
    }
    C* d = s + __mul24(gg * N + m, pitch) + j3;
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * (M * pitch)] = v[r];
  }
}

// axis 2, inverse pass a, to the planes in memory
template <int N, int S, bool STREAM, typename C>
__device__ __forceinline__ void ax2_store(const C* s, C* dst, int n3, int pitch, int gc, const C* tw) {
  constexpr int A = radix_a(N), R = A > 1 ? A : N, M = N / R;
  const int mn = M * n3, total = gc * mn;
  const float rmn = rcp_of(mn), r3 = rcp_of(n3);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int gg = gc > 1 ? fdiv(idx, rmn) : 0, rem = idx - __mul24(gg, mn);
    const int m = M > 1 ? fdiv(rem, r3) : 0, j3 = rem - __mul24(m, n3);
    const C* p = s + __mul24(gg * N + m, pitch) + j3;
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = p[r * (M * pitch)];
    if constexpr (M > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = cmul(v[r], twid<S>(tw[(r - 1) * M + m]));
    }
    Dft<R, S, C>::run(v);
    const unsigned o = static_cast<unsigned>(__mul24(gg, N * n3) + rem) * sizeof(C);
#pragma unroll
    for (int r = 0; r < R; ++r) stream_store<STREAM>(lane_at(dst + r * mn, o), v[r]);
  }
}

// axis 2, pass b
template <int N, int S, typename C>
__device__ __forceinline__ void ax2_b(C* s, int n3, int pitch, int gc) {
  constexpr int A = radix_a(N), R = N / A;
  const int total = gc * A * n3;
  const float r3 = rcp_of(n3);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int gk = fdiv(idx, r3), j3 = idx - __mul24(gk, n3);
    C* p = s + __mul24(gk * R, pitch) + j3;
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = p[r * pitch];
    Dft<R, S, C>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) p[r * pitch] = v[r];
  }
}

// axis 3: consecutive lanes take consecutive rows, whose pitch N | 1 is odd,
// so the lanes spread over all LDS banks
// pass a (INV: backwards, twiddles before the DFT)
template <int N, int S, bool INV, typename C>
__device__ __forceinline__ void ax3_a(C* s, int rows, const C* tw) {
  constexpr int R = radix_a(N), M = N / R, P = N | 1;
  const int total = rows * M;
  const float rr = rcp_of(rows);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int j = fdiv(idx, rr), row = idx - __mul24(j, rows);
    C* p = s + __mul24(row, P) + j;
    const C* w = tw + j;
    C v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[r] = p[r * M];
      if (INV && r > 0) v[r] = cmul(v[r], twid<S>(w[(r - 1) * M]));
    }
    Dft<R, S, C>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) p[r * M] = !INV && r > 0 ? cmul(v[r], twid<S>(w[(r - 1) * M])) : v[r];
  }
}

// axis 3, pass b (or the only pass)
template <int N, int S, typename C>
__device__ __forceinline__ void ax3_b(C* s, int rows) {
  constexpr int A = radix_a(N), R = N / A, P = N | 1;
  const int total = rows * A;
  const float rr = rcp_of(rows);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int k1 = fdiv(idx, rr), row = idx - __mul24(k1, rows);
    C* p = s + __mul24(row, P) + k1 * R;
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
template <int N, bool EN, bool BACK, typename C, typename T>
__device__ __forceinline__ void ax3_kernel(C* s, int rows, const T* __restrict__ v, double* en) {
  constexpr int A = radix_a(N), R = N / A, P = N | 1;
  const int total = rows * A;
  const float rr = rcp_of(rows);
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int k1 = fdiv(idx, rr), row = idx - __mul24(k1, rows);
    T vv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) vv[r] = *lane_at(v + r * total, static_cast<unsigned>(idx) * sizeof(T));
    C* p = s + __mul24(row, P) + k1 * R;
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
