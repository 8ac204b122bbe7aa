// FFT building blocks for gfx950: complex helpers, in-register DFTs of the
// small radices, the factorisation of a line and the twiddle tables.
//
// Lengths: every {2,3,5}-smooth L in [2, 72].  Twiddles come from a per-L
// table W_L^t = exp(-2 pi i t / L) built in FP64 on the host and rounded once
// to the working precision.
#pragma once

#include <hip/hip_runtime.h>

namespace fock {

constexpr int kNMax = 72;   // largest supported grid axis
constexpr int kBlock = 256; // threads per workgroup of the fills and reductions

// ---------------------------------------------------------------------------
// complex helpers on HIP vector types (x = real, y = imaginary)
// ---------------------------------------------------------------------------
template <typename T> struct cx;
template <> struct cx<float> { using t = float2; };
template <> struct cx<double> { using t = double2; };

template <typename C> __device__ __forceinline__ C cadd(C a, C b) { return C{a.x + b.x, a.y + b.y}; }
template <typename C> __device__ __forceinline__ C csub(C a, C b) { return C{a.x - b.x, a.y - b.y}; }
template <typename C> __device__ __forceinline__ C cmul(C a, C b) {
  return C{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename C> __device__ __forceinline__ C cmulconj(C a, C b) {  // conj(a) * b
  return C{a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x};
}
template <typename C, typename S> __device__ __forceinline__ C cscale(C a, S s) { return C{a.x * s, a.y * s}; }
// multiply by s*i with s = +1 or -1
template <int S, typename C> __device__ __forceinline__ C cmul_si(C a) {
  return S > 0 ? C{-a.y, a.x} : C{a.y, -a.x};
}

// ---------------------------------------------------------------------------
// in-register DFTs, X[k] = sum_n x[n] exp(S * 2 pi i n k / R), S = -1 forward
// ---------------------------------------------------------------------------
template <int R, int S, typename C> struct Dft;

template <int S, typename C> struct Dft<2, S, C> {
  static __device__ __forceinline__ void run(C* x) {
    C a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
  }
};

template <int S, typename C> struct Dft<3, S, C> {
  static __device__ __forceinline__ void run(C* x) {
    using T = decltype(x[0].x);
    const T h = T(0.8660254037844386467637231707529362);  // sin(2 pi / 3)
    C t1 = cadd(x[1], x[2]);
    C t2 = csub(x[1], x[2]);
    C m = C{x[0].x - T(0.5) * t1.x, x[0].y - T(0.5) * t1.y};
    C r = cmul_si<S>(cscale(t2, h));
    x[0] = cadd(x[0], t1);
    x[1] = cadd(m, r);
    x[2] = csub(m, r);
  }
};

template <int S, typename C> struct Dft<4, S, C> {
  static __device__ __forceinline__ void run(C* x) {
    C a = cadd(x[0], x[2]), b = csub(x[0], x[2]);
    C c = cadd(x[1], x[3]), d = cmul_si<S>(csub(x[1], x[3]));
    x[0] = cadd(a, c);
    x[2] = csub(a, c);
    x[1] = cadd(b, d);
    x[3] = csub(b, d);
  }
};

template <int S, typename C> struct Dft<5, S, C> {
  static __device__ __forceinline__ void run(C* x) {
    using T = decltype(x[0].x);
    const T c1 = T(0.3090169943749474241022934171828191);   // cos(2 pi / 5)
    const T c2 = T(-0.8090169943749474241022934171828191);  // cos(4 pi / 5)
    const T s1 = T(0.9510565162951535721164393333793821);   // sin(2 pi / 5)
    const T s2 = T(0.5877852522924731291687059546390728);   // sin(4 pi / 5)
    C a1 = cadd(x[1], x[4]), b1 = csub(x[1], x[4]);
    C a2 = cadd(x[2], x[3]), b2 = csub(x[2], x[3]);
    C x0 = x[0];
    C m1 = C{x0.x + c1 * a1.x + c2 * a2.x, x0.y + c1 * a1.y + c2 * a2.y};
    C m2 = C{x0.x + c2 * a1.x + c1 * a2.x, x0.y + c2 * a1.y + c1 * a2.y};
    C n1 = cmul_si<S>(C{s1 * b1.x + s2 * b2.x, s1 * b1.y + s2 * b2.y});
    C n2 = cmul_si<S>(C{s2 * b1.x - s1 * b2.x, s2 * b1.y - s1 * b2.y});
    x[0] = cadd(x0, cadd(a1, a2));
    x[1] = cadd(m1, n1);
    x[4] = csub(m1, n1);
    x[2] = cadd(m2, n2);
    x[3] = csub(m2, n2);
  }
};

template <int S, typename C> struct Dft<8, S, C> {
  // two length-4 DFTs over even and odd inputs, combined with w8^k
  static __device__ __forceinline__ void run(C* x) {
    using T = decltype(x[0].x);
    const T r2 = T(0.7071067811865475244008443621048490);  // 1/sqrt(2)
    C e[4] = {x[0], x[2], x[4], x[6]};
    C o[4] = {x[1], x[3], x[5], x[7]};
    Dft<4, S, C>::run(e);
    Dft<4, S, C>::run(o);
    // w8^1 = (1 + S i)/sqrt2, w8^2 = S i, w8^3 = (-1 + S i)/sqrt2
    C o1 = cscale(cadd(o[1], cmul_si<S>(o[1])), r2);
    C o2 = cmul_si<S>(o[2]);
    C o3 = cscale(csub(cmul_si<S>(o[3]), o[3]), r2);
    x[0] = cadd(e[0], o[0]);
    x[4] = csub(e[0], o[0]);
    x[1] = cadd(e[1], o1);
    x[5] = csub(e[1], o1);
    x[2] = cadd(e[2], o2);
    x[6] = csub(e[2], o2);
    x[3] = cadd(e[3], o3);
    x[7] = csub(e[3], o3);
  }
};

// ---------------------------------------------------------------------------
// compile-time factorisation
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int pick_radix(int rem) {
  return rem % 8 == 0 ? 8 : rem % 4 == 0 ? 4 : rem % 2 == 0 ? 2 : rem % 3 == 0 ? 3 : 5;
}

__host__ __device__ constexpr bool smooth235(int n) {
  if (n < 1) return false;
  while (n % 2 == 0) n /= 2;
  while (n % 3 == 0) n /= 3;
  while (n % 5 == 0) n /= 5;
  return n == 1;
}

// Twiddle tables of every supported length, concatenated in increasing L.
__host__ __device__ constexpr int twiddle_offset(int L) {
  int off = 0;
  for (int n = 2; n < L; ++n)
    if (smooth235(n)) off += n;
  return off;
}
constexpr int kTwiddleTotal = twiddle_offset(kNMax + 1);

// fast quotient for idx < 2^20 and any n >= 1: the fractional part of
// (idx + 0.5)/n stays >= 0.5/n away from an integer, and the FP32 error of
// the product is at most 3 2^-24 idx/n, less than 0.19/n.
__device__ __forceinline__ int fdiv(int idx, float rcp) {
  return static_cast<int>((static_cast<float>(idx) + 0.5f) * rcp);
}

}  // namespace fock
