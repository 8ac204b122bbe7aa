// The three-pass kernels of the exchange (paper, "Our Implementation": the
// band-pair loop that runs on the GPU; "CPU Performance Analysis": FFTs, data
// manipulation and the accumulate that make up FOCK_ACC), for any
// {2,3,5}-smooth axes up to 72, and the batched 3-D DFT.
//
// The pair buffer keeps the grid's own order, T[c1][j2][j3], and only axis 1,
// the one with the largest stride, is transformed in registers (reg_fft.hpp):
//
//   forward  thread (j2, j3): rho = conj(u_m) u_n along axis 1, FFT_1 -> T
//   plane    workgroup (pair, planes of fixed c1): FFT_2, FFT_3, x v_q/N (the
//            pair energies), IFFT_3, IFFT_2, all in LDS (plane_fft.hpp)
//   acc      thread (j2, j3): for every partner of the batch IFFT_1 of its
//            line of T, acc += -w' f' u_m W in registers; one write (or add)
//            of the output per batch
//
// So the first and the last pass are compiled for one axis length and take
// the other two at run time, their loads are contiguous over the whole plane
// whatever its shape, and the accumulate, which runs once per ordered pair,
// has one transform of the six and no LDS.  Lines too long for a lane's
// registers live in a lane pair (split_fft.hpp).
//
// Every pass is meant to be bound by the pair buffer's traffic: one write, one
// read and write, two reads (one per order of a pair).  At 32^3 4x4x4 k, 18
// bands, FP64 (7.7 GB a batch) the passes take 1.73, 2.87 and 2.67 ms: 4.5, 5.4
// and 5.8 TB/s, a large copy's 4.9 to 5.4.
//
// It serves FP64 plans on every grid and V_x of FP32 plans on general grids
// (FP32 N1 x L x L and mixed plans: pass_reg.hip; why, and FP32 energies:
// energy_lds.hip).  Against the passes it replaced, per call.  All transforms
// in LDS with a barrier around every radix pass, ordered pairs (general grids):
// 24x24x60, 3x3x1 k, 12 bands, FP32 step 27.8 -> 9.0 ms; 36x40x45, 2x1x1 k, 16
// bands, FP64 apply 4.55 -> 0.60 ms; 160 DFTs of 48^3 FP64 498 -> 300 us.  Plane
// transforms over whole register lines (N1 x L x L): 60^3 Gamma FP64 2.00 ->
// 1.35 ms; 32^3 2x2x2 k FP64 step 11.3 -> 10.0; apply with energy at Gamma FP64:
// 24x72x72 1.64 -> 0.76, 36^3 1.14 -> 0.72, 60x40x40 1.00 -> 0.72, 72x24x24 0.89
// -> 0.88 ms.
#include <algorithm>

#include "fft_lds.hpp"
#include "fock_internal.hpp"
#include "pass_common.hpp"
#include "plane_fft.hpp"
#include "reg_fft.hpp"
#include "split_fft.hpp"

namespace fock {

// A line of L in one lane, or half of it in each lane of a pair where line
// (and accumulator) would take more registers than half a SIMD's.
template <typename T, int L>
struct LineShape {
  static constexpr int REGS = L * static_cast<int>(2 * sizeof(T)) / 4;
  static constexpr bool FP32 = sizeof(T) == 4;
  static constexpr bool SPLIT_FWD = L % 2 == 0 && REGS > 144;
  // the accumulate over lane pairs: always, or (FP32 54 and 72 points) where a
  // lane per line leaves the chip short of waves
  static constexpr bool SPLIT_ACC = L % 2 == 0 && (FP32 ? L == 48 || L == 50 || L == 60 || L == 64 : REGS > 80);
  static constexpr bool SPLIT_ACC_FEW = FP32 && (L == 54 || L == 72);
  static constexpr int FWD_REGS = SPLIT_FWD ? REGS / 2 : REGS;
  // waves per SIMD (register budget 512 / WPE)
  static constexpr int WPE_FWD = FWD_REGS <= 144 ? 2 : 1;
};

template <typename T, int L, bool SPLIT>
struct AccShape {
  static constexpr int REGS = LineShape<T, L>::REGS / (SPLIT ? 2 : 1);
  // three waves per SIMD for FP64 where 168 registers hold them: 32^3 2x2x2 k
  // step 10.41 -> 10.05 ms (FP32 loses: 32^3 4x4x4 k on this path, as with
  // FOCK_NO_REG=1, 336.0 -> 341.6 ms)
  static constexpr int WPE = sizeof(T) == 8 && 2 * REGS <= 128 ? 3 : 2 * REGS <= 160 ? 2 : 1;
  // most waves of a workgroup: two per SIMD, or what 64 KiB of LDS take of their sums
  static constexpr int BYTES = REGS * 64 * 4;
  static constexpr int WAVES0 = 64 * 1024 / BYTES + 1;
  static constexpr int WAVES1 = WPE >= 2 ? 8 : 4;
  static constexpr int WAVES = WAVES0 < WAVES1 ? WAVES0 : WAVES1;
};

// Item of workgroup b when `total` items are dealt to the eight XCDs in
// contiguous runs (workgroups go to the XCDs in turn): neighbouring items,
// which share orbital slices, then share an L2.  >= total: no item.
__device__ __forceinline__ unsigned xcd_item(unsigned b, unsigned total) {
  return (b & 7u) * ((total + 7u) >> 3) + (b >> 3);
}
inline unsigned xcd_grid(unsigned total) { return ((total + 7u) >> 3) * 8u; }

// x[j] = conj(b[j * stride]) a[j * stride] at the lane's byte offset o (a and
// b wave-uniform): a straight into the line (all loads in flight at once),
// then b in batches multiplied in place, so that only two batches of operands
// are live beside the line.
template <typename C, int L>
__device__ __forceinline__ void load_codensity_u(C* x, const C* __restrict__ a, const C* __restrict__ b, unsigned o,
                                                 size_t stride) {
  constexpr int B = batch_of(L, kRegB);
  constexpr int NB = L / B;
#pragma unroll
  for (int j = 0; j < L; ++j) x[j] = *lane_at(a + j * stride, o);
  C bb[2][B];
#pragma unroll
  for (int j = 0; j < B; ++j) bb[0][j] = *lane_at(b + j * stride, o);
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    if (n + 1 < NB) {
#pragma unroll
      for (int j = 0; j < B; ++j) bb[(n + 1) & 1][j] = *lane_at(b + ((n + 1) * B + j) * stride, o);
    }
    reg_fence();
#pragma unroll
    for (int j = 0; j < B; ++j) x[n * B + j] = cmulconj(bb[n & 1][j], x[n * B + j]);
  }
}

// ---------------------------------------------------------------------------
// forward pass: rho = conj(u_m) u_n, FFT along axis 1, T[c1][j2][j3]
// ---------------------------------------------------------------------------
// Items (line block, pair), pairs fastest; pairs not null: the explicit pair
// list of an energy batch.  The pass writes the pair buffer once and should
// read orbitals from L2 only, so a line block is one wave: the slices of a
// batch's 128 partners (32^3: 16 KB each) then stay in an XCD's 4 MB while it
// walks the pairs; four waves' slices (8 MB) come from further away.  32^3
// 4x4x4 k FP32 on this path (FOCK_NO_REG=1), 3.9 GB a batch: 1060 us at four
// waves, 730 at one (5.3 TB/s).
template <typename T, int L, bool STREAM>
__global__ __launch_bounds__(64, (LineShape<T, L>::WPE_FWD)) void k_line_fwd(
    int plane, int npairs, unsigned total, int nbands, long long bs, const typename cx<T>::t* __restrict__ psi, int o0,
    int nP, int tri, const int2* __restrict__ parts, const PairRef* __restrict__ pairs,
    typename cx<T>::t* __restrict__ tbuf) {
  using C = typename cx<T>::t;
  constexpr bool SPLIT = LineShape<T, L>::SPLIT_FWD;
  constexpr int LN = SPLIT ? L / 2 : L;
  const unsigned it = xcd_item(blockIdx.x, total);
  if (it >= total) return;
  const int lb = it / npairs, pi = it - lb * npairs;
  const int id = lb * 64 + static_cast<int>(threadIdx.x);
  const int l = SPLIT ? id >> 1 : id, h = SPLIT ? id & 1 : 0;
  if (l >= plane) return;  // both lanes of a pair together; no barrier in this kernel
  int okn, pkm;
  if (pairs) {
    const PairRef pr = pairs[pi];
    okn = pr.k * nbands + pr.n;
    pkm = pr.kp * nbands + pr.m;
  } else {
    int o, p;
    batch_pair(pi, nP, tri, &o, &p);
    okn = o0 + o;
    const int2 r = parts[p];
    pkm = r.x * nbands + r.y;
  }
  C x[LN];
  const unsigned lo = (static_cast<unsigned>(h) * plane + l) * sizeof(C);  // split: samples j1 = 2m + h
  load_codensity_u<C, LN>(x, psi + static_cast<size_t>(okn) * bs, psi + static_cast<size_t>(pkm) * bs, lo,
                          static_cast<size_t>(SPLIT ? 2 : 1) * plane);
  if constexpr (SPLIT)
    split_fft_fwd<C, L>(x, h);  // x[k] at c1 = h L/2 + k
  else
    reg_fft<C, L, -1>(x);
  C* base = tbuf + static_cast<size_t>(pi) * plane * L;
  const unsigned so = opaque((static_cast<unsigned>(h) * LN * plane + l) * sizeof(C));
#pragma unroll
  for (int k = 0; k < LN; ++k) lane_store<STREAM>(base + static_cast<size_t>(k) * plane, so, x[k]);
}

// ---------------------------------------------------------------------------
// plane pass: axes 2 and 3 forward, x v_q/N, and back, in place
// ---------------------------------------------------------------------------
// EN: the weighted pair energies into epart[pair * tiles + tile]; BACK: the
// inverse transforms (an energy batch has no way back).
// What the pass has to do is one read and one write of the tile; the rest are
// six LDS round trips of the values.
template <typename T, bool EN, bool BACK, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_plane_pair(PlaneGeo g, int nbands, int nk, int o0, int nP, int tri,
                                                        const int2* __restrict__ parts, const int* __restrict__ qmap,
                                                        const PairRef* __restrict__ pairs,
                                                        typename cx<T>::t* tbuf,
                                                        const T* __restrict__ vtab,
                                                        const typename cx<T>::t* __restrict__ tw2,
                                                        const typename cx<T>::t* __restrict__ tw3,
                                                        const double* __restrict__ occ, const double* __restrict__ kw,
                                                        double* __restrict__ epart) {
  using C = typename cx<T>::t;
  extern __shared__ unsigned char smem_raw[];
  C* t2 = reinterpret_cast<C*>(smem_raw);  // twiddles of the two axes, then the tile
  C* t3 = t2 + g.tw2;
  C* s = t3 + g.tw3;
  const int pi = blockIdx.x, tile = blockIdx.y, g0 = tile * g.g, gc = min(g.g, g.n1 - g0);
  const int plane = g.n2 * g.n3, rows = gc * g.n2;
  int q;
  double w = 1.0;
  if constexpr (BACK) {
    int o, p;
    batch_pair(pi, nP, tri, &o, &p);
    const int ok = (o0 + o) / nbands;
    const int2 r = parts[p];
    q = qmap[ok * nk + r.x];
    // an unordered pair of a block with itself stands for both orders
    if constexpr (EN) w = (tri && o != p ? 2.0 : 1.0) * kw[ok] * occ[o0 + o] * kw[r.x] * occ[r.x * nbands + r.y];
  } else {
    const PairRef pr = pairs[pi];
    q = pr.q;
    w = pr.mult * kw[pr.k] * occ[pr.k * nbands + pr.n] * kw[pr.kp] * occ[pr.kp * nbands + pr.m];
  }
  for (int i = threadIdx.x; i < g.tw2 + g.tw3; i += blockDim.x) t2[i] = i < g.tw2 ? tw2[i] : tw3[i - g.tw2];
  const size_t at = (static_cast<size_t>(pi) * g.n1 + g0) * plane;
  const T* v = vtab + (static_cast<size_t>(q) * g.n1 + g0) * plane;
  double e = 0.0;
  switch (g.n2) {
#define CASE(N)                                              \
  case N:                                                    \
    ax2_load<N, -1, STREAM>(s, tbuf + at, g.n3, g.pitch, gc, tw2); \
    __syncthreads();                                         \
    if constexpr (radix_a(N) > 1) {                          \
      ax2_b<N, -1, C>(s, g.n3, g.pitch, gc);                 \
      __syncthreads();                                       \
    }                                                        \
    break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
  }
  switch (g.n3) {
#define CASE(N)                                              \
  case N:                                                    \
    if constexpr (radix_a(N) > 1) {                          \
      ax3_a<N, -1, false, C>(s, rows, t3);                   \
      __syncthreads();                                       \
    }                                                        \
    ax3_kernel<N, EN, BACK, C, T>(s, rows, v, &e);           \
    if constexpr (BACK && radix_a(N) > 1) {                  \
      __syncthreads();                                       \
      ax3_a<N, +1, true, C>(s, rows, t3);                    \
    }                                                        \
    break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
  }
  if constexpr (BACK) {
    __syncthreads();
    switch (g.n2) {
#define CASE(N)                                              \
  case N:                                                    \
    if constexpr (radix_a(N) > 1) {                          \
      ax2_b<N, +1, C>(s, g.n3, g.pitch, gc);                 \
      __syncthreads();                                       \
    }                                                        \
    ax2_store<N, +1, STREAM>(s, tbuf + at, g.n3, g.pitch, gc, t2); \
    break;
      FOCK_SMOOTH_L(CASE)
#undef CASE
    }
  }
  if constexpr (EN) {  // fixed order: across the lanes, then the waves in turn
    __shared__ double red[8];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
      double sum = 0.0;
      for (unsigned i = 0; i < blockDim.x / 64; ++i) sum += red[i];
      epart[static_cast<size_t>(pi) * gridDim.y + tile] = w * sum;
    }
  }
}

// ---------------------------------------------------------------------------
// accumulate pass (rows and partners as in acc_source)
// ---------------------------------------------------------------------------
// One workgroup per item (line block, row), rows fastest: the workgroups of one
// line block, which read the same slices of the partners' orbitals at about
// the same time, run on one XCD and take them from its L2.  Its waves share
// the row's partners out in contiguous slices and their sums meet in LDS in
// order: where lines and rows are few, a chain of one partner after another in
// one wave is what the pass takes (two memory latencies each).
// Once they do, loading a partner's orbital together with its pair gains no
// more (the batch of twelve cells 834 -> 822 us, 12x10x9 53.0 -> 54.6).
template <typename T, int L, bool SPLIT, bool STREAM>
__global__ __launch_bounds__((AccShape<T, L, SPLIT>::WAVES * 64), (AccShape<T, L, SPLIT>::WPE)) void k_line_acc(
    int plane, int rows, unsigned total, int nbands, long long bs, int o0, int nO, int nP, int tri,
    const int2* __restrict__ parts, const typename cx<T>::t* __restrict__ tbuf,
    const typename cx<T>::t* __restrict__ psi, const double* __restrict__ occ, const double* __restrict__ kw,
    typename cx<T>::t* __restrict__ out, int first, int first_mirror, const double* __restrict__ gscale, double hscale,
    int backward) {
  using C = typename cx<T>::t;
  constexpr int LN = SPLIT ? L / 2 : L;
  constexpr int B = batch_of(LN, AccShape<T, L, SPLIT>::WPE == 1 ? 16 : kRegB);
  constexpr int NB = LN / B;
  extern __shared__ unsigned char smem_raw[];
  const unsigned it = xcd_item(blockIdx.x, total);
  if (it >= total) return;  // the whole workgroup
  const int lb = it / rows, row = it - lb * rows;
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int id = lb * 64 + lane;
  const int lv = SPLIT ? id >> 1 : id, h = SPLIT ? id & 1 : 0;
  const int l = min(lv, plane - 1);  // lanes past the plane repeat its last line and store nothing
  const bool mirror = row >= nO;
  const int o = mirror ? row - nO : row;
  const int nsrc = mirror ? nO : nP;
  const unsigned lt = (static_cast<unsigned>(h) * LN * plane + l) * sizeof(C);  // split: c1 = h L/2 + k
  const unsigned lu = (static_cast<unsigned>(h) * plane + l) * sizeof(C);       // split: j1 = 2m + h
  const size_t us = static_cast<size_t>(SPLIT ? 2 : 1) * plane;
  C acc[LN];
#pragma unroll
  for (int j = 0; j < LN; ++j) acc[j] = C{T(0), T(0)};
  const int p1 = (wave + 1) * nsrc / nw;
  for (int p = wave * nsrc / nw; p < p1; ++p) {
    int sb;
    size_t pair;
    bool cj;
    acc_source(mirror, p, o, o0, nP, tri, nbands, parts, &sb, &pair, &cj);
    const C* src = tbuf + pair * plane * L;
    // copies made here: an offset from outside the loop would be widened there
    // and added to the base for every element
    const unsigned ot = opaque(lt), ou = opaque(lu);
    C x[LN];
#pragma unroll
    for (int k = 0; k < LN; ++k) x[k] = lane_load<STREAM>(src + static_cast<size_t>(k) * plane, ot);
    if constexpr (SPLIT)
      split_fft_inv<C, L>(x, h);
    else
      reg_fft<C, L, +1>(x);
    if (cj) {
#pragma unroll
      for (int j = 0; j < LN; ++j) x[j].y = -x[j].y;
    }
    const T coef = static_cast<T>(-kw[sb / nbands] * occ[sb]);
    const C* um = psi + static_cast<size_t>(sb) * bs;
    C mb[2][B];
#pragma unroll
    for (int j = 0; j < B; ++j) mb[0][j] = lane_load(um + j * us, ou);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if (n + 1 < NB) {
#pragma unroll
        for (int j = 0; j < B; ++j) mb[(n + 1) & 1][j] = lane_load(um + ((n + 1) * B + j) * us, ou);
      }
      reg_fence();
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const C w = cmul(mb[n & 1][j], x[n * B + j]);
        acc[n * B + j].x += coef * w.x;
        acc[n * B + j].y += coef * w.y;
      }
    }
  }
  if (nw > 1) {
    C* s = reinterpret_cast<C*>(smem_raw) + lane;  // [wave - 1][j][lane]
    if (wave > 0) {
#pragma unroll
      for (int j = 0; j < LN; ++j) s[((wave - 1) * LN + j) * 64] = acc[j];
    }
    __syncthreads();
    if (wave > 0) return;
    for (int w = 1; w < nw; ++w) {
#pragma unroll
      for (int j = 0; j < LN; ++j) acc[j] = cadd(acc[j], s[((w - 1) * LN + j) * 64]);
    }
  }
  if (lv >= plane) return;
  const int okn = mirror ? parts[o].x * nbands + parts[o].y : o0 + o;
  double f = hscale;
  if (gscale) f *= gscale[0];
  if (backward) f *= kw[okn / nbands] * occ[okn];
  const T ft = static_cast<T>(f);
  C* dst = out + static_cast<size_t>(okn) * bs;
  const unsigned ou = opaque(lu);
  if (!(mirror ? first_mirror : first)) {
    // loaded before the first store, so the loads overlap
    C old[LN];
#pragma unroll
    for (int j = 0; j < LN; ++j) old[j] = lane_load(dst + j * us, ou);
#pragma unroll
    for (int j = 0; j < LN; ++j) lane_store(dst + j * us, ou, cadd(old[j], cscale(acc[j], ft)));
  } else {
#pragma unroll
    for (int j = 0; j < LN; ++j) lane_store(dst + j * us, ou, cscale(acc[j], ft));
  }
}

// ---------------------------------------------------------------------------
// plain batched 3-D DFT in the natural layout
// ---------------------------------------------------------------------------
// axis 1 of line (j2, j3) = l, coalesced across lanes
template <typename T, int L, int S>
__global__ __launch_bounds__(256, (LineShape<T, L>::WPE_FWD)) void k_dft_line(int plane,
                                                                              typename cx<T>::t* __restrict__ data,
                                                                              long long stride) {
  using C = typename cx<T>::t;
  constexpr bool SPLIT = LineShape<T, L>::SPLIT_FWD;
  constexpr int LN = SPLIT ? L / 2 : L;
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  const int l = SPLIT ? id >> 1 : id, h = SPLIT ? id & 1 : 0;
  if (l >= plane) return;
  C* d = data + static_cast<size_t>(blockIdx.y) * stride;
  // split lines: samples 2m + h and half spectra h L/2 + k, in the order the transform takes and gives
  const unsigned eo = (static_cast<unsigned>(h) * plane + l) * sizeof(C);
  const unsigned hf = (static_cast<unsigned>(h) * LN * plane + l) * sizeof(C);
  const size_t s1 = static_cast<size_t>(plane), s2 = static_cast<size_t>(SPLIT ? 2 : 1) * plane;
  C x[LN];
#pragma unroll
  for (int j = 0; j < LN; ++j) x[j] = lane_load(d + j * (S < 0 ? s2 : s1), S < 0 ? eo : hf);
  if constexpr (!SPLIT)
    reg_fft<C, L, S>(x);
  else if constexpr (S < 0)
    split_fft_fwd<C, L>(x, h);
  else
    split_fft_inv<C, L>(x, h);
  const unsigned so = opaque(S < 0 ? hf : eo);
#pragma unroll
  for (int j = 0; j < LN; ++j) lane_store(d + j * (S < 0 ? s1 : s2), so, x[j]);
}

// axes 2 and 3 of a tile of planes; the frequencies leave LDS in order
template <typename T, int S>
__global__ __launch_bounds__(512, 4) void k_dft_plane(PlaneGeo g, typename cx<T>::t* __restrict__ data, long long stride,
                                                      const typename cx<T>::t* __restrict__ tw2,
                                                      const typename cx<T>::t* __restrict__ tw3) {
  using C = typename cx<T>::t;
  extern __shared__ unsigned char smem_raw[];
  C* t3 = reinterpret_cast<C*>(smem_raw);
  C* s = t3 + g.tw3;
  const int g0 = blockIdx.x * g.g, gc = min(g.g, g.n1 - g0);
  const int plane = g.n2 * g.n3, rows = gc * g.n2;
  for (int i = threadIdx.x; i < g.tw3; i += blockDim.x) t3[i] = tw3[i];
  C* t = data + static_cast<size_t>(blockIdx.y) * stride + static_cast<size_t>(g0) * plane;
  switch (g.n2) {
#define CASE(N)                                              \
  case N:                                                    \
    ax2_load<N, S, false>(s, t, g.n3, g.pitch, gc, tw2);     \
    if constexpr (radix_a(N) > 1) {                          \
      __syncthreads();                                       \
      ax2_b<N, S, C>(s, g.n3, g.pitch, gc);                  \
    }                                                        \
    break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
  }
  __syncthreads();
  switch (g.n3) {
#define CASE(N)                                              \
  case N:                                                    \
    if constexpr (radix_a(N) > 1) {                          \
      ax3_a<N, S, false, C>(s, rows, t3);                    \
      __syncthreads();                                       \
    }                                                        \
    ax3_b<N, S, C>(s, rows);                                 \
    break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
  }
  __syncthreads();
  const float r3 = rcp_of(g.n3), r2 = rcp_of(g.n2), ra2 = rcp_of(g.a2), ra3 = rcp_of(g.a3);
  for (int e = threadIdx.x; e < gc * plane; e += blockDim.x) {
    const int row = fdiv(e, r3), c3 = e - row * g.n3;
    const int gg = fdiv(row, r2), c2 = row - gg * g.n2;
    const int k2 = fdiv(c2, ra2), k3 = fdiv(c3, ra3);  // c = (c mod a) + a k at position (c mod a) b + k
    t[e] = s[(gg * g.n2 + (c2 - k2 * g.a2) * g.b2 + k2) * g.pitch + (c3 - k3 * g.a3) * g.b3 + k3];
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

size_t plane_lds(const PlaneGeo& g, size_t csize) {
  return (static_cast<size_t>(g.g) * g.n2 * g.pitch + g.tw2 + g.tw3) * csize;
}

template <typename T, int L>
void line_fwd_L(const Plan& p, const Batch& b, const Instance& in, const void* psi, const int2* parts,
                const PairRef* pairs, typename cx<T>::t* tbuf) {
  const int plane = in.grid[1] * in.grid[2];
  const int lanes = plane * (LineShape<T, L>::SPLIT_FWD ? 2 : 1);
  const unsigned total = static_cast<unsigned>((lanes + 63) / 64) * b.npairs;
  by_stream(p, b, [&](auto stream) {
    hipLaunchKernelGGL((k_line_fwd<T, L, stream()>), dim3(xcd_grid(total)), dim3(64), 0, p.stream, plane, b.npairs,
                       total, in.nbands, static_cast<long long>(in.band_stride),
                       static_cast<const typename cx<T>::t*>(psi), b.o0, b.nP, b.tri, parts, pairs, tbuf);
  });
}

template <typename T, int L, bool SPLIT>
void line_acc_launch(const Plan& p, const Batch& b, const Instance& in, const int2* parts,
                     const typename cx<T>::t* tbuf, const void* psi, const double* occ, const double* kw, void* out,
                     const double* gscale, double hscale, bool backward) {
  using C = typename cx<T>::t;
  using Sh = AccShape<T, L, SPLIT>;
  const int plane = in.grid[1] * in.grid[2];
  const int lanes = plane * (SPLIT ? 2 : 1);
  const int rows = b.nO + (b.mirror ? b.nP : 0);
  const unsigned total = static_cast<unsigned>((lanes + 63) / 64) * rows;
  // Partners shared out among waves while that leaves at most 4096 waves in all
  // (the chip holds 2048 to 8192) and two partners to a wave.  One wave per
  // row and line block, sharing up to 2048 waves, up to 4096: batch of twelve
  // cells (288 to 600 waves a launch) 1203, 834, 822 us; 12x10x9 step (12
  // waves) 59, 53, 53; 36x40x45 FP64 apply (1824 waves) 793, 792, 779.
  const int nsrc = b.mirror ? std::min(b.nO, b.nP) : b.nP;
  int nw = 1;
  while (nw < Sh::WAVES && total * static_cast<unsigned>(nw + 1) <= 4096u && 2 * (nw + 1) <= nsrc) ++nw;
  const size_t lds = static_cast<size_t>(nw - 1) * Sh::BYTES;
  by_stream(p, b, [&](auto stream) {
    hipLaunchKernelGGL((k_line_acc<T, L, SPLIT, stream()>), dim3(xcd_grid(total)), dim3(64 * nw), lds, p.stream, plane,
                       rows, total, in.nbands, static_cast<long long>(in.band_stride), b.o0, b.nO, b.nP, b.tri, parts,
                       tbuf, static_cast<const C*>(psi), occ, kw, static_cast<C*>(out), b.first, b.first_mirror, gscale,
                       hscale, backward ? 1 : 0);
  });
}

template <typename T, int L>
void line_acc_L(const Plan& p, const Batch& b, const Instance& in, const int2* parts, const typename cx<T>::t* tbuf,
                const void* psi, const double* occ, const double* kw, void* out, const double* gscale, double hscale,
                bool backward) {
  using Sh = LineShape<T, L>;
  if constexpr (Sh::SPLIT_ACC_FEW) {
    // Apply, lane pairs against whole lines, on this path (FOCK_NO_REG=1): 72^3
    // FP32, 20 bands (1620 waves of whole lines) 0.79 against 0.81 ms, 72x24x24,
    // 60 bands (540) 0.75 against 0.82; 72^3, 64 bands (5184) 7.84 against 7.73
    const long long waves =
        static_cast<long long>((in.grid[1] * in.grid[2] + 63) / 64) * (b.nO + (b.mirror ? b.nP : 0));
    if (waves <= 2048) {
      line_acc_launch<T, L, true>(p, b, in, parts, tbuf, psi, occ, kw, out, gscale, hscale, backward);
      return;
    }
  }
  line_acc_launch<T, L, Sh::SPLIT_ACC>(p, b, in, parts, tbuf, psi, occ, kw, out, gscale, hscale, backward);
}

template <typename T>
hipError_t line_fwd(const Plan& p, const Batch& b, const Instance& in, const void* psi, const int2* parts,
                    const PairRef* pairs, typename cx<T>::t* tbuf) {
  switch (in.grid[0]) {
#define CASE(N) \
  case N: line_fwd_L<T, N>(p, b, in, psi, parts, pairs, tbuf); break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t line_apply_t(const Plan& p, const Batch& b, const void* psi, const double* occ, void* out,
                        const double* gscale, double hscale, bool backward, bool energy) {
  using C = typename cx<T>::t;
  const Instance& in = p.inst[b.inst];
  const PlaneGeo& g = in.pg;
  const int2* parts = reinterpret_cast<const int2*>(p.ws + b.part_off);
  const int* qmap = reinterpret_cast<const int*>(p.ws + in.qmap_off);
  const T* vtab = reinterpret_cast<const T*>(p.ws + in.vtab_off);
  const double* kw = reinterpret_cast<const double*>(p.ws + in.kw_off);
  const C* tw = reinterpret_cast<const C*>(p.ws + p.tw_off);
  C* tbuf = reinterpret_cast<C*>(p.ws + p.tbuf_off);
  double* epart = reinterpret_cast<double*>(p.ws + p.epart_off);
  p.prof.begin(FOCK_K_PLANE, p.stream);
  hipError_t e = line_fwd<T>(p, b, in, psi, parts, nullptr, tbuf);
  p.prof.end(FOCK_K_PLANE, p.stream);
  if (e != hipSuccess) return e;
  const int tiles = plane_tiles(g);
  const dim3 grid(b.npairs, tiles);
  const C *tw2 = tw + twiddle_offset(g.n2), *tw3 = tw + twiddle_offset(g.n3);
  p.prof.begin(FOCK_K_PENCIL, p.stream);
  if constexpr (sizeof(T) == 4) energy = false;  // energy_lds.hip
  constexpr bool EN = sizeof(T) == 8;
  by_stream(p, b, [&](auto stream) {
    if (energy)
      hipLaunchKernelGGL((k_plane_pair<T, EN, true, stream()>), grid, dim3(in.pg_threads), plane_lds(g, sizeof(C)),
                         p.stream, g, in.nbands, in.nk, b.o0, b.nP, b.tri, parts, qmap,
                         static_cast<const PairRef*>(nullptr), tbuf, vtab, tw2, tw3, occ, kw, epart);
    else
      hipLaunchKernelGGL((k_plane_pair<T, false, true, stream()>), grid, dim3(in.pg_threads), plane_lds(g, sizeof(C)),
                         p.stream, g, in.nbands, in.nk, b.o0, b.nP, b.tri, parts, qmap,
                         static_cast<const PairRef*>(nullptr), tbuf, vtab, tw2, tw3, occ, kw, epart);
  });
  p.prof.end(FOCK_K_PENCIL, p.stream);
  if (energy) {
    e = launch_sum_slot(p, static_cast<long long>(b.npairs) * tiles, b.eslot, b.mirror ? 2.0 : 1.0);
    if (e != hipSuccess) return e;
  }
  p.prof.begin(FOCK_K_ACCUMULATE, p.stream);
  switch (g.n1) {
#define CASE(N) \
  case N: line_acc_L<T, N>(p, b, in, parts, tbuf, psi, occ, kw, out, gscale, hscale, backward); break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  p.prof.end(FOCK_K_ACCUMULATE, p.stream);
  return hipGetLastError();
}

hipError_t line_energy(const Plan& p, const Batch& b, const void* psi, const double* occ) {
  using T = double;
  using C = typename cx<T>::t;
  const Instance& in = p.inst[b.inst];
  const PlaneGeo& g = in.pg;
  const PairRef* pairs = reinterpret_cast<const PairRef*>(p.ws + b.pair_off);
  const C* tw = reinterpret_cast<const C*>(p.ws + p.tw_off);
  C* tbuf = reinterpret_cast<C*>(p.ws + p.tbuf_off);
  p.prof.begin(FOCK_K_ENERGY_PLANE, p.stream);
  const hipError_t e = line_fwd<T>(p, b, in, psi, nullptr, pairs, tbuf);
  p.prof.end(FOCK_K_ENERGY_PLANE, p.stream);
  if (e != hipSuccess) return e;
  const int tiles = plane_tiles(g);
  p.prof.begin(FOCK_K_ENERGY_PENCIL, p.stream);
  by_stream(p, b, [&](auto stream) {
    hipLaunchKernelGGL((k_plane_pair<T, true, false, stream()>), dim3(b.npairs, tiles), dim3(in.pg_threads),
                       plane_lds(g, sizeof(C)), p.stream, g, in.nbands, in.nk, 0, 1, 0,
                       static_cast<const int2*>(nullptr), static_cast<const int*>(nullptr), pairs, tbuf,
                       reinterpret_cast<const T*>(p.ws + in.vtab_off),
                       tw + twiddle_offset(g.n2), tw + twiddle_offset(g.n3), occ,
                       reinterpret_cast<const double*>(p.ws + in.kw_off),
                       reinterpret_cast<double*>(p.ws + p.epart_off));
  });
  p.prof.end(FOCK_K_ENERGY_PENCIL, p.stream);
  return launch_sum_slot(p, static_cast<long long>(b.npairs) * tiles, b.slot, 1.0);
}

template <typename T, int L, int S>
void dft_line_L(const Plan& p, int plane, int count, typename cx<T>::t* d, long long stride) {
  const int lanes = plane * (LineShape<T, L>::SPLIT_FWD ? 2 : 1);
  const int nt = std::min(256, (lanes + 63) / 64 * 64);
  hipLaunchKernelGGL((k_dft_line<T, L, S>), dim3((lanes + nt - 1) / nt, count), dim3(nt), 0, p.stream, plane, d, stride);
}

template <typename T, int S>
hipError_t line_dft3_t(const Plan& p, const PlaneGeo& g, int threads, int count, void* data, long long stride) {
  using C = typename cx<T>::t;
  C* d = static_cast<C*>(data);
  const C* tw = reinterpret_cast<const C*>(p.ws + p.tw_off);
  hipLaunchKernelGGL((k_dft_plane<T, S>), dim3(plane_tiles(g), count), dim3(threads), plane_lds(g, sizeof(C)),
                     p.stream, g, d, stride, tw + twiddle_offset(g.n2), tw + twiddle_offset(g.n3));
  switch (g.n1) {
#define CASE(N) \
  case N: dft_line_L<T, N, S>(p, g.n2 * g.n3, count, d, stride); break;
    FOCK_SMOOTH_L(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
void plane_lds_attr(int lim) {
  constexpr bool EN = sizeof(T) == 8;  // FP32 energies: energy_lds.hip
  const void* fs[] = {reinterpret_cast<const void*>(&k_plane_pair<T, false, true, false>),
                      reinterpret_cast<const void*>(&k_plane_pair<T, false, true, true>),
                      reinterpret_cast<const void*>(&k_plane_pair<T, EN, true, false>),
                      reinterpret_cast<const void*>(&k_plane_pair<T, EN, true, true>),
                      reinterpret_cast<const void*>(&k_plane_pair<T, EN, !EN, false>),
                      reinterpret_cast<const void*>(&k_plane_pair<T, EN, !EN, true>),
                      reinterpret_cast<const void*>(&k_dft_plane<T, -1>),
                      reinterpret_cast<const void*>(&k_dft_plane<T, +1>)};
  for (const void* f : fs)
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lim) != hipSuccess) (void)hipGetLastError();
}

}  // namespace

int plane_tiles(const PlaneGeo& g) { return (g.n1 + g.g - 1) / g.g; }

size_t plane_lds_bytes(const PlaneGeo& g, size_t csize) { return plane_lds(g, csize); }

static int plane_threads(const PlaneGeo& g) {
  const int pts = g.g * g.n2 * g.n3;
  return pts >= 3200 ? 512 : pts >= 1440 ? 256 : pts >= 1050 ? 192 : pts >= 500 ? 128 : 64;
}

// Tile and workgroup of the plane passes, from sweeps of both on eleven plane
// sizes (256 to 5184 points) in both precisions.
//   Tile: whole planes of up to 2880 points in FP32, 1440 in FP64 (23 KB of LDS:
//   seven tiles a compute unit; one larger plane is a tile by itself), but
//   several planes only while that leaves 1024 workgroups.  24x60 FP32: two
//   planes 276 us, one 293; 40x40 FP32: one 261, two 264; 40x40 FP64 249, 264.
//   Threads: five to eleven points each, and a multiple of four waves where the
//   tile gives them: 320 or 384 threads leave the SIMDs unevenly filled.
//   40x40 FP32: 256 threads 261 us, 320 323, 384 353, 192 262, 128 270; 48x48
//   FP64: 256 247, 384 286; 72x72 FP64: 512 449, 384 475, 256 525.
void plane_geometry(const int grid[3], long long planes_of, size_t csize, int max_tiles, PlaneGeo* g, int* threads) {
  g->n1 = grid[0];
  g->n2 = grid[1];
  g->n3 = grid[2];
  g->a2 = radix_a(g->n2);
  g->b2 = g->n2 / g->a2;
  g->a3 = radix_a(g->n3);
  g->b3 = g->n3 / g->a3;
  g->tw2 = twiddle_count(g->n2);
  g->tw3 = twiddle_count(g->n3);
  g->pitch = g->n3 | 1;
  g->g = std::max(1, std::min(g->n1, (csize == 16 ? 1440 : 2880) / (g->n2 * g->n3)));
  while (g->g > 1 && planes_of * plane_tiles(*g) < 1024) g->g = (g->g + 1) / 2;
  g->g = std::max(g->g, (g->n1 + max_tiles - 1) / max_tiles);
  *threads = plane_threads(*g);
}

hipError_t launch_apply_batch(const Plan& p, const Batch& b, const void* psi, const double* occ, void* out,
                              bool energy, const double* gscale, double hscale, bool backward) {
  if (p.inst[b.inst].reg) return launch_reg_apply_batch(p, b, psi, occ, out, gscale, hscale, backward, energy);
  return p.prec == FOCK_C64
             ? line_apply_t<float>(p, b, psi, occ, out, gscale, hscale, backward, energy)
             : line_apply_t<double>(p, b, psi, occ, out, gscale, hscale, backward, energy);
}

hipError_t launch_energy_batch(const Plan& p, const Batch& b, const void* psi, const double* occ) {
  if (p.inst[b.inst].reg) return launch_reg_energy_batch(p, b, psi, occ);
  return p.prec == FOCK_C64 ? launch_lds_energy_batch(p, b, psi, occ, nullptr)
                            : line_energy(p, b, psi, occ);
}

hipError_t launch_line_dft3(const Plan& p, int inst, int sign, int count, void* data, long long stride) {
  const Instance& in = p.inst[inst];
  // Tiles of at most 256 points where planes are small (the plan's are for its
  // pairs): 16384 DFTs of 16^3 FP32 377 us with one plane a tile, 424 with 11.
  PlaneGeo g = in.pg;
  g.g = std::max(1, std::min(g.n1, 256 / (g.n2 * g.n3)));
  const int threads = plane_threads(g);
  if (p.io64())
    return sign < 0 ? line_dft3_t<double, -1>(p, g, threads, count, data, stride)
                    : line_dft3_t<double, +1>(p, g, threads, count, data, stride);
  return sign < 0 ? line_dft3_t<float, -1>(p, g, threads, count, data, stride)
                  : line_dft3_t<float, +1>(p, g, threads, count, data, stride);
}

void prepare_line_kernels(fock_precision prec, int lim) {
  if (prec == FOCK_C64) {
    plane_lds_attr<float>(lim);
    return;
  }
  plane_lds_attr<double>(lim);
}

}  // namespace fock
