// E_x of FP32 plans on general grids: all transforms in LDS, one radix pass
// after another over a plane (axes 3 and 2) and a slab (axis 1), FP64 sums.
//
// An energy is an FP64 number made of FP32 spectra, and other transform forms
// round those differently: taken from the plane pass of pass_line.hip, E_x moves
// by up to 6e-8 of itself (either form repeats bit for bit and is as far from the
// FP64 value, within 1e-6).  It keeps this form, over ordered pairs after an
// apply and over unordered ones in fock_energy, so that the energies of one input
// agree to 1e-12 with those that the library gave before V_x took the faster
// passes.  24x24x60, 3x3x1 k, 12 bands, FP32 step: 28.0 ms when V_x took this
// form too, 9.0 with E_x alone in it, 3.4 with E_x from the plane pass.
#include <algorithm>

#include "fft_lds.hpp"
#include "fock_internal.hpp"
#include "plane_fft.hpp"

namespace fock {

struct Geo {
  int n1, n2, n3;
  int nk, nbands;
  long long bs;  // band stride in elements
};

// ---------------------------------------------------------------------------
// one Stockham pass of radix R over `nlines` lines of length L in LDS.
// ROWS: elements of a line are contiguous (estride 1) and consecutive lanes
// take consecutive butterflies of one line; otherwise lines are contiguous
// (lstride 1) and consecutive lanes take consecutive lines.
// ---------------------------------------------------------------------------
template <typename C, int L, int R, int NS, int S, bool ROWS>
__device__ __forceinline__ void stockham_pass(C* s, int nlines, float rcp_lines, int lstride, int estride,
                                              const C* __restrict__ tw) {
  constexpr int M = L / R;
  constexpr int MAXB = (kNMax * M + kBlock - 1) / kBlock;
  const int nbf = nlines * M;
  C v[MAXB][R];
#pragma unroll
  for (int b = 0; b < MAXB; ++b) {
    const int idx = static_cast<int>(threadIdx.x) + b * kBlock;
    if (idx < nbf) {
      int line, j;
      if (ROWS) {
        line = idx / M;
        j = idx - line * M;
      } else {
        j = fdiv(idx, rcp_lines);
        line = idx - j * nlines;
      }
      const C* src = s + line * lstride;
      const int k = j % NS;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        C x = src[(j + r * M) * estride];
        if (NS > 1 && r > 0) {
          C w = tw[r * k * (L / (NS * R))];
          if (S > 0) w.y = -w.y;
          x = cmul(x, w);
        }
        v[b][r] = x;
      }
      Dft<R, S, C>::run(v[b]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < MAXB; ++b) {
    const int idx = static_cast<int>(threadIdx.x) + b * kBlock;
    if (idx < nbf) {
      int line, j;
      if (ROWS) {
        line = idx / M;
        j = idx - line * M;
      } else {
        j = fdiv(idx, rcp_lines);
        line = idx - j * nlines;
      }
      C* dst = s + line * lstride;
      const int k = j % NS;
      const int d = (j / NS) * NS * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) dst[(d + r * NS) * estride] = v[b][r];
    }
  }
  __syncthreads();
}

template <typename C, int L, int NS, int S, bool ROWS>
__device__ __forceinline__ void stockham_passes(C* s, int nlines, float rcp_lines, int lstride, int estride,
                                                const C* __restrict__ tw) {
  if constexpr (NS < L) {
    constexpr int R = pick_radix(L / NS);
    stockham_pass<C, L, R, NS, S, ROWS>(s, nlines, rcp_lines, lstride, estride, tw);
    stockham_passes<C, L, NS * R, S, ROWS>(s, nlines, rcp_lines, lstride, estride, tw);
  }
}

// Transform `nlines` lines of runtime length L (a supported size) in LDS.
// `twall` is the concatenated twiddle table.  Must be called by all threads.
template <typename C, int S, bool ROWS>
__device__ __forceinline__ void fft_lines(C* s, int L, int nlines, int lstride, int estride,
                                       const C* __restrict__ twall) {
  const float rcp = 1.0f / static_cast<float>(nlines);
#define FOCK_FFT_CASE(LL)                                                                  \
  case LL:                                                                                 \
    stockham_passes<C, LL, 1, S, ROWS>(s, nlines, rcp, lstride, estride, twall + twiddle_offset(LL)); \
    break;
  switch (L) {
    FOCK_FFT_CASE(2) FOCK_FFT_CASE(3) FOCK_FFT_CASE(4) FOCK_FFT_CASE(5) FOCK_FFT_CASE(6)
    FOCK_FFT_CASE(8) FOCK_FFT_CASE(9) FOCK_FFT_CASE(10) FOCK_FFT_CASE(12) FOCK_FFT_CASE(15)
    FOCK_FFT_CASE(16) FOCK_FFT_CASE(18) FOCK_FFT_CASE(20) FOCK_FFT_CASE(24) FOCK_FFT_CASE(25)
    FOCK_FFT_CASE(27) FOCK_FFT_CASE(30) FOCK_FFT_CASE(32) FOCK_FFT_CASE(36) FOCK_FFT_CASE(40)
    FOCK_FFT_CASE(45) FOCK_FFT_CASE(48) FOCK_FFT_CASE(50) FOCK_FFT_CASE(54) FOCK_FFT_CASE(60)
    FOCK_FFT_CASE(64) FOCK_FFT_CASE(72)
    default:
      break;  // unreachable: the planner admits supported lengths only
  }
#undef FOCK_FFT_CASE
}

// plane pass: rho = conj(u_m) u_n, axes 3 and 2 forward, per (pair, j1)
template <typename T, bool EXPLICIT>
__global__ __launch_bounds__(kBlock) void k_fwd_plane(Geo g, const typename cx<T>::t* __restrict__ psi, int o0,
                                                      int nP, const int2* __restrict__ parts,
                                                      const PairRef* __restrict__ pairs,
                                                      typename cx<T>::t* __restrict__ tbuf,
                                                      const typename cx<T>::t* __restrict__ tw) {
  using C = typename cx<T>::t;
  extern __shared__ unsigned char smem_raw[];
  C* s = reinterpret_cast<C*>(smem_raw);
  const int j1 = blockIdx.x, pi = blockIdx.y;
  int okn, pkm;  // global band indices k*nbands + n
  if (EXPLICIT) {
    const PairRef pr = pairs[pi];
    okn = pr.k * g.nbands + pr.n;
    pkm = pr.kp * g.nbands + pr.m;
  } else {
    const int o = pi / nP, p = pi - o * nP;
    okn = o0 + o;
    const int2 r = parts[p];
    pkm = r.x * g.nbands + r.y;
  }
  const int plane = g.n2 * g.n3;
  const C* a = psi + static_cast<size_t>(okn) * g.bs + static_cast<size_t>(j1) * plane;
  const C* b = psi + static_cast<size_t>(pkm) * g.bs + static_cast<size_t>(j1) * plane;
  for (int e = threadIdx.x; e < plane; e += kBlock) s[e] = cmulconj(b[e], a[e]);
  __syncthreads();
  fft_lines<C, -1, true>(s, g.n3, g.n2, g.n3, 1, tw);   // axis 3 (rows)
  fft_lines<C, -1, false>(s, g.n2, g.n3, 1, g.n3, tw);  // axis 2 (columns)
  C* t = tbuf + (static_cast<size_t>(pi) * g.n1 + j1) * plane;
  for (int e = threadIdx.x; e < plane; e += kBlock) t[e] = s[e];
}

// Offset of class (c1, c2, c3) in a kernel table stored in the order of the
// plane passes (plan.cpp).
__device__ __forceinline__ int table_at(const PlaneGeo& g, int c1, int c2, int c3) {
  const int g0 = c1 / g.g * g.g, rows = min(g.g, g.n1 - g0) * g.n2;
  const int q2 = c2 / g.a2;
  return g0 * g.n2 * g.n3 + c3 * rows + (c1 - g0) * g.n2 + (c2 - q2 * g.a2) * g.b2 + q2;
}

// pencil pass: axis 1 of slab c2 and sum_c v_q(c)/N |P(c)|^2 in FP64, weighted if
// occ is given.  EXPLICIT: a pair list; otherwise the ordered pairs of a batch.  vtab
// is in grid order (one load of n3 values after another), or, where the plan has
// no room for that, the plane passes' table (tiled; 24x24x60, 528 pairs: 66.4
// -> 88.9 us).
template <typename T, bool EXPLICIT>
__global__ __launch_bounds__(kBlock) void k_pencil_energy(Geo g, PlaneGeo pg, int tiled, int o0, int nP,
                                                          const int2* __restrict__ parts, const int* __restrict__ qmap,
                                                          const PairRef* __restrict__ pairs,
                                                          const typename cx<T>::t* __restrict__ tbuf,
                                                          const T* __restrict__ vtab,
                                                          const typename cx<T>::t* __restrict__ tw,
                                                          const double* __restrict__ occ,
                                                          const double* __restrict__ kw, double* __restrict__ epart,
                                                          unsigned* done, double* __restrict__ ex, double factor) {
  using C = typename cx<T>::t;
  extern __shared__ unsigned char smem_raw[];
  __shared__ double red[kBlock / 64];
  C* s = reinterpret_cast<C*>(smem_raw);
  const int c2 = blockIdx.x, pi = blockIdx.y;
  int q;
  double w = 1.0;
  if constexpr (EXPLICIT) {
    const PairRef pr = pairs[pi];
    q = pr.q;
    if (occ) w = kw[pr.k] * occ[pr.k * g.nbands + pr.n] * kw[pr.kp] * occ[pr.kp * g.nbands + pr.m];
  } else {
    const int o = pi / nP, p = pi - o * nP, ok = (o0 + o) / g.nbands;
    const int2 r = parts[p];
    q = qmap[ok * g.nk + r.x];
    w = kw[ok] * occ[o0 + o] * kw[r.x] * occ[r.x * g.nbands + r.y];
  }
  const int plane = g.n2 * g.n3, tile = g.n1 * g.n3;
  const size_t npts = static_cast<size_t>(g.n1) * plane;
  const C* base = tbuf + static_cast<size_t>(pi) * npts + static_cast<size_t>(c2) * g.n3;
  const float rcp3 = 1.0f / static_cast<float>(g.n3);
  for (int e = threadIdx.x; e < tile; e += kBlock) {
    const int j1 = fdiv(e, rcp3), c3 = e - j1 * g.n3;
    s[e] = base[static_cast<size_t>(j1) * plane + c3];
  }
  __syncthreads();
  fft_lines<C, -1, false>(s, g.n1, g.n3, 1, g.n3, tw);
  const T* v = vtab + static_cast<size_t>(q) * npts;
  double acc = 0.0;
  for (int e = threadIdx.x; e < tile; e += kBlock) {
    const int c1 = fdiv(e, rcp3), c3 = e - c1 * g.n3;
    const double px = static_cast<double>(s[e].x), py = static_cast<double>(s[e].y);
    const int at = tiled ? table_at(pg, c1, c2, c3) : (c1 * g.n2 + c2) * g.n3 + c3;
    acc += static_cast<double>(v[at]) * (px * px + py * py);
  }
  const double tot = block_sum(acc, red);
  if (threadIdx.x == 0) epart[static_cast<size_t>(pi) * g.n2 + c2] = w * tot;
  if (!ex) return;
  // The workgroup that ends last sums the partials, compensated and in a fixed
  // order, and clears the counter for the next launch.
  __shared__ bool last;
  const unsigned n = gridDim.x * gridDim.y;
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
  __syncthreads();
  if (!last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  double sum = 0.0, comp = 0.0;
  for (unsigned i = threadIdx.x; i < n; i += kBlock) neumaier(sum, comp, epart[i]);
  const double all = block_sum(sum + comp, red);
  if (threadIdx.x == 0) {
    ex[0] = factor * all;
    *done = 0u;
  }
}

// Small batches after an apply: the pencil pass sums its partials, without the
// launch of the sum, and where every instance has one such batch finishes E_x,
// without k_energy_finish's too.  Every workgroup then waits for its partial to
// leave the L2, with what else it holds, which past some 300 workgroups or 20000
// points takes as long as the launches.  Apply and E_x at Gamma, with those launches /
// without, us: 4x4x4, 2 bands 28.3/25.4; four instances, by partials of each, 8^3, 3
// bands (72) 98.7/83.5, 4x4x4, 8 bands (256) 100/88, 5x8x6, 6 bands (288) 99/100, 8^3, 8
// bands (512) 101/116; by points, 12x10x9, 4 bands (17280) 99/95, 5 bands (27000)
// 101/112, 10x4x20, 9 bands (64800) 110/131.
static bool finishes(const Instance& in, const Batch& b) {
  const long long pairs = b.npairs;
  return pairs * in.grid[1] <= 288 && pairs * in.npts <= 20480;
}

bool lds_energy_whole(const Plan& p) {
  if (p.ordered_energy.size() != p.inst.size()) return false;
  for (const Batch& b : p.ordered_energy) {
    const Instance& in = p.inst[b.inst];
    if (in.n_aslot != 1 || !finishes(in, b)) return false;
  }
  return true;
}

// After an apply (b.eslot >= 0): the ordered pairs of a batch, or of a list that
// holds those of several groups, weighted, into slot b.eslot, or E_x if ex is
// given.  Else a list of fock_energy, into slot b.slot.
hipError_t launch_lds_energy_batch(const Plan& p, const Batch& b, const void* psi, const double* occ, double* ex) {
  using C = float2;
  const Instance& in = p.inst[b.inst];
  const Geo g{in.grid[0], in.grid[1], in.grid[2], in.nk, in.nbands, static_cast<long long>(in.band_stride)};
  const C* tw = reinterpret_cast<const C*>(p.ws + p.tw1_off);
  const int2* parts = reinterpret_cast<const int2*>(p.ws + b.part_off);
  const PairRef* pairs = reinterpret_cast<const PairRef*>(p.ws + b.pair_off);
  const int* qmap = reinterpret_cast<const int*>(p.ws + in.qmap_off);
  const float* vtab = reinterpret_cast<const float*>(p.ws + in.etab_off);
  const int tiled = in.etab_off == in.vtab_off;
  unsigned* done = reinterpret_cast<unsigned*>(p.ws + p.tw1_off + static_cast<size_t>(kTwiddleTotal) * sizeof(C));
  const double* kw = reinterpret_cast<const double*>(p.ws + in.kw_off);
  C* tbuf = reinterpret_cast<C*>(p.ws + p.tbuf_off);
  double* epart = reinterpret_cast<double*>(p.ws + p.epart_off);
  const size_t lds_plane = static_cast<size_t>(g.n2) * g.n3 * sizeof(C);
  const size_t lds_tile = static_cast<size_t>(g.n1) * g.n3 * sizeof(C);
  const bool ordered = b.nO > 0, after = b.eslot >= 0;
  const double factor = ex ? energy_factor(in) : 1.0;
  if (!ex && after && finishes(in, b)) ex = reinterpret_cast<double*>(p.ws + p.ebsum_off) + b.eslot;
  p.prof.begin(FOCK_K_ENERGY_PLANE, p.stream);
  if (ordered)
    hipLaunchKernelGGL((k_fwd_plane<float, false>), dim3(g.n1, b.npairs), dim3(kBlock), lds_plane, p.stream, g,
                       static_cast<const C*>(psi), b.o0, b.nP, parts, static_cast<const PairRef*>(nullptr), tbuf, tw);
  else
    hipLaunchKernelGGL((k_fwd_plane<float, true>), dim3(g.n1, b.npairs), dim3(kBlock), lds_plane, p.stream, g,
                       static_cast<const C*>(psi), 0, 1, static_cast<const int2*>(nullptr), pairs, tbuf, tw);
  p.prof.end(FOCK_K_ENERGY_PLANE, p.stream);
  p.prof.begin(FOCK_K_ENERGY_PENCIL, p.stream);
  if (ordered)
    hipLaunchKernelGGL((k_pencil_energy<float, false>), dim3(g.n2, b.npairs), dim3(kBlock), lds_tile, p.stream, g,
                       in.pg, tiled, b.o0, b.nP, parts, qmap, static_cast<const PairRef*>(nullptr),
                       static_cast<const C*>(tbuf), vtab, tw, occ, kw, epart, done, ex, factor);
  else
    hipLaunchKernelGGL((k_pencil_energy<float, true>), dim3(g.n2, b.npairs), dim3(kBlock), lds_tile, p.stream, g,
                       in.pg, tiled, 0, 1, static_cast<const int2*>(nullptr), static_cast<const int*>(nullptr), pairs,
                       static_cast<const C*>(tbuf), vtab, tw, after ? occ : nullptr, kw, epart, done, ex,
                       factor);
  p.prof.end(FOCK_K_ENERGY_PENCIL, p.stream);
  if (ex) return hipGetLastError();
  if (after) return launch_sum_slot(p, static_cast<long long>(b.npairs) * g.n2, b.eslot, 1.0);
  return launch_energy_reduce(p, b, occ, g.n2);
}

}  // namespace fock
