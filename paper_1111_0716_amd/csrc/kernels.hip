// Reductions and fills of the exchange hot path for gfx950, and the dispatch
// of a batch to its path's kernels.
//
// Energies: per (pair, tile) partial sums in FP64, then a fixed-order tree per
// batch and a compensated (Neumaier) sum over batches.
#include <algorithm>

#include "fft_lds.hpp"
#include "fock_internal.hpp"
#include "pass_common.hpp"

namespace fock {

// ---------------------------------------------------------------------------
// energy reductions
// ---------------------------------------------------------------------------
// one workgroup per energy batch: sum_c2 per pair, weight, fixed-order tree
__global__ __launch_bounds__(kBlock) void k_energy_batch(const PairRef* __restrict__ pairs, int npairs, int n2,
                                                         const double* __restrict__ epart,
                                                         const double* __restrict__ occ,
                                                         const double* __restrict__ kw, int nbands,
                                                         double* __restrict__ ebsum, int slot) {
  __shared__ double red[kBlock / 64];
  double sum = 0.0, comp = 0.0;
  for (int pi = threadIdx.x; pi < npairs; pi += kBlock) {
    const PairRef pr = pairs[pi];
    double e = 0.0;
    for (int c = 0; c < n2; ++c) e += epart[static_cast<size_t>(pi) * n2 + c];
    const double w = pr.mult * kw[pr.k] * occ[pr.k * nbands + pr.n] * kw[pr.kp] * occ[pr.kp * nbands + pr.m];
    const double x = w * e;
    neumaier(sum, comp, x);
  }
  const double tot = block_sum(sum + comp, red);
  if (threadIdx.x == 0) ebsum[slot] = tot;
}

// slots[slot] = mult * (sum of part[0..n)) in a fixed order: Neumaier per
// thread over a strided share, then the waves in order (1024 threads: the
// partials of a batch run to hundreds of thousands, read once, eight loads in
// flight: 141264 partials took 75 us one at a time, 70632 take 14).  mult is 2 for a batch of
// unordered pairs (each stands for both orders), else 1.
constexpr int kSumBlock = 1024;
__global__ __launch_bounds__(kSumBlock) void k_sum_slot(const double* __restrict__ part, long long n,
                                                        double* __restrict__ slots, int slot, double mult) {
  __shared__ double red[kSumBlock / 64];
  double sum = 0.0, comp = 0.0;
  for (long long i0 = threadIdx.x; i0 < n; i0 += 8 * kSumBlock) {
    double x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = i0 + u * kSumBlock < n ? part[i0 + u * kSumBlock] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) neumaier(sum, comp, x[u]);
  }
  double v = sum + comp;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kSumBlock / 64; ++w) t += red[w];
    slots[slot] = mult * t;
  }
}

// ex[i] = factor * (sum of src[0 .. count)) in order, a workgroup for each
// instance of the launch (one launch for each costs a few us apiece).  Its
// lanes load 64 values at once and hand them on in turn (a load for each value
// in turn is a memory latency per value: 32 partials 3.5 -> 3.2 us).
struct FinishItem {
  const double* src;
  double factor;
  int count;
};
// N: instances a launch has room for; one by itself, since a launch takes longer
// by its arguments' size (E_x of 4x4x4 20.7 us with 64, 20.2 with one).
constexpr int kFinishItems = 64;
template <int N>
struct FinishArgs {
  FinishItem it[N];
};
template <int N>
__global__ __launch_bounds__(64) void k_energy_finish(const FinishArgs<N> args, double* __restrict__ ex) {
  const FinishItem& in = args.it[blockIdx.x];
  double sum = 0.0, comp = 0.0;
  for (int i0 = 0; i0 < in.count; i0 += 64) {
    const int i = i0 + static_cast<int>(threadIdx.x);
    const double mine = i < in.count ? in.src[i] : 0.0;
    const int n = min(64, in.count - i0);
    for (int u = 0; u < n; ++u) neumaier(sum, comp, __shfl(mine, u, 64));
  }
  if (threadIdx.x == 0) ex[blockIdx.x] = in.factor * (sum + comp);
}

// ---------------------------------------------------------------------------
// zero the outputs of k-points that have no partner in the k-pair list
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_zero_bands(typename cx<T>::t* __restrict__ out, int b0, long long bs,
                                                       long long npts) {
  using C = typename cx<T>::t;
  C* dst = out + static_cast<size_t>(b0 + blockIdx.y) * bs;
  for (long long e = blockIdx.x * static_cast<long long>(kBlock) + threadIdx.x; e < npts;
       e += static_cast<long long>(gridDim.x) * kBlock)
    dst[e] = C{T(0), T(0)};
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

template <typename T>
hipError_t zero_outputs_t(const Plan& p, int inst, void* out) {
  using C = typename cx<T>::t;
  const Instance& in = p.inst[inst];
  for (int k = 0; k < in.nk; ++k) {
    if (!in.kpartners[k].empty()) continue;
    const int gx = static_cast<int>(std::min<long long>(1024, (in.npts + kBlock - 1) / kBlock));
    p.prof.begin(FOCK_K_OTHER, p.stream);
    hipLaunchKernelGGL((k_zero_bands<T>), dim3(gx, in.nbands), dim3(kBlock), 0, p.stream, static_cast<C*>(out),
                       k * in.nbands, static_cast<long long>(in.band_stride), static_cast<long long>(in.npts));
    p.prof.end(FOCK_K_OTHER, p.stream);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_zero_all_bands(const Plan& p, int inst, void* out) {
  const Instance& in = p.inst[inst];
  const int gx = static_cast<int>(std::min<long long>(1024, (in.npts + kBlock - 1) / kBlock));
  const int nbt = in.nk * in.nbands;
  for (int b0 = 0; b0 < nbt; b0 += 65535) {
    const int nb = std::min(65535, nbt - b0);
    p.prof.begin(FOCK_K_OTHER, p.stream);
    if (p.io64()) {
      hipLaunchKernelGGL((k_zero_bands<double>), dim3(gx, nb), dim3(kBlock), 0, p.stream, static_cast<double2*>(out),
                         b0, static_cast<long long>(in.band_stride), static_cast<long long>(in.npts));
    } else {
      hipLaunchKernelGGL((k_zero_bands<float>), dim3(gx, nb), dim3(kBlock), 0, p.stream, static_cast<float2*>(out),
                         b0, static_cast<long long>(in.band_stride), static_cast<long long>(in.npts));
    }
    p.prof.end(FOCK_K_OTHER, p.stream);
  }
  return hipGetLastError();
}

hipError_t launch_zero_outputs(const Plan& p, int inst, void* out) {
  return p.io64() ? zero_outputs_t<double>(p, inst, out) : zero_outputs_t<float>(p, inst, out);
}

hipError_t prepare_kernels(fock_precision prec, size_t* max_lds) {
  int dev = 0, lim = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  if (e != hipSuccess) return e;
  *max_lds = static_cast<size_t>(lim);
  prepare_fused_kernels(prec, lim - 256);
  prepare_reg_kernels(prec, lim - 64);
  prepare_line_kernels(prec, lim - 64);
  return hipSuccess;
}

hipError_t launch_energy_reduce(const Plan& p, const Batch& b, const double* occ, int n2) {
  const Instance& in = p.inst[b.inst];
  p.prof.begin(FOCK_K_ENERGY_REDUCE, p.stream);
  hipLaunchKernelGGL(k_energy_batch, dim3(1), dim3(kBlock), 0, p.stream,
                     reinterpret_cast<const PairRef*>(p.ws + b.pair_off), b.npairs, n2,
                     reinterpret_cast<const double*>(p.ws + p.epart_off), occ,
                     reinterpret_cast<const double*>(p.ws + in.kw_off), in.nbands,
                     reinterpret_cast<double*>(p.ws + p.ebsum_off), b.slot);
  p.prof.end(FOCK_K_ENERGY_REDUCE, p.stream);
  return hipGetLastError();
}

hipError_t launch_sum_slot(const Plan& p, long long n, int slot, double mult) {
  p.prof.begin(FOCK_K_ENERGY_REDUCE, p.stream);
  hipLaunchKernelGGL(k_sum_slot, dim3(1), dim3(kSumBlock), 0, p.stream, reinterpret_cast<const double*>(p.ws + p.epart_off),
                     n, reinterpret_cast<double*>(p.ws + p.ebsum_off), slot, mult);
  p.prof.end(FOCK_K_ENERGY_REDUCE, p.stream);
  return hipGetLastError();
}

hipError_t launch_sum_partials(const Plan& p, const double* part, long long n, int slot) {
  p.prof.begin(FOCK_K_ENERGY_REDUCE, p.stream);
  hipLaunchKernelGGL(k_sum_slot, dim3(1), dim3(kSumBlock), 0, p.stream, part, n,
                     reinterpret_cast<double*>(p.ws + p.ebsum_off), slot, 1.0);
  p.prof.end(FOCK_K_ENERGY_REDUCE, p.stream);
  return hipGetLastError();
}

hipError_t launch_energy_finish(const Plan& p, double* ex, bool after_apply) {
  const double* slots = reinterpret_cast<const double*>(p.ws + p.ebsum_off);
  const double* eblk = reinterpret_cast<const double*>(p.ws + p.eblk_off);
  const int n = static_cast<int>(p.inst.size());
  for (int i0 = 0; i0 < n; i0 += kFinishItems) {
    const int m = std::min(kFinishItems, n - i0);
    FinishArgs<kFinishItems> a{};
    for (int j = 0; j < m; ++j) {
      const Instance& in = p.inst[i0 + j];
      FinishItem& t = a.it[j];
      t.factor = energy_factor(in);
      if (!after_apply) {
        t.src = slots + in.first_ebatch;
        t.count = in.n_ebatches;
      } else if (!in.fused) {
        t.src = slots + in.first_aslot;
        t.count = in.n_aslot;
      } else if (in.rounds >= 0) {
        // one partial per unordered pair: summed in a fixed order into the
        // instance's slot first
        const FusedRounds& r = p.fused_rounds[in.rounds];
        const hipError_t e = launch_sum_partials(p, eblk + r.eblk0, r.npairs, r.eslot);
        if (e != hipSuccess) return e;
        t.src = slots + r.eslot;
        t.count = 1;
      } else {
        t.src = eblk + in.first_eblk;
        t.count = in.n_eblk;
      }
    }
    p.prof.begin(FOCK_K_ENERGY_REDUCE, p.stream);
    if (m == 1)
      hipLaunchKernelGGL(k_energy_finish<1>, dim3(1), dim3(64), 0, p.stream, FinishArgs<1>{{a.it[0]}}, ex + i0);
    else
      hipLaunchKernelGGL(k_energy_finish<kFinishItems>, dim3(m), dim3(64), 0, p.stream, a, ex + i0);
    p.prof.end(FOCK_K_ENERGY_REDUCE, p.stream);
  }
  return hipGetLastError();
}

}  // namespace fock
