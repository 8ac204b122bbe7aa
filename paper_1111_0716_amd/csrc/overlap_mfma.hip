// Band overlap M[k][i][j] = dV sum_e conj(u_{k,i}[e]) (V_x u)_{k,j}[e] on the
// matrix cores (the dense contraction on the path; paper, "CPU Performance
// Analysis": the BLAS share of FOCK).
//
// A complex N_b x N_b product over K = N grid points, split over K chunks.
// One workgroup of four waves owns a 32 x 32 block of M (four 16 x 16
// tiles, one per wave) over one chunk: the 32 bands of u and the 32 bands of
// V_x u of the block are staged through LDS a slab of kSlab grid points at a
// time (16-byte loads, two slabs in flight), so each operand element read
// from memory serves two tiles.  Each wave multiplies its tile with 16x16x4
// MFMA instructions, four real products per complex step
// (Re += ar br + ai bi, Im += ar bi - ai br), and writes its chunk partial in
// FP64; a second kernel sums the chunk partials in a fixed order and applies
// dV.
//
// Operand layout of the 16x16x4 instruction (both precisions): lane l gives
// A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16]; it receives
// D[i][j = l % 16] for v = 0..3 with i = 4 (l / 16) + v (FP32) or
// i = l / 16 + 4 v (FP64), as measured on gfx950.
#include <algorithm>
#include <type_traits>

#include "fock_internal.hpp"
#include "fft_lds.hpp"

namespace fock {

namespace {

constexpr int kOvWaves = 4;
constexpr int kOvSub = 1024;    // points accumulated in the MFMA precision before an FP64 fold
constexpr int kBlk = 32;        // bands per block side (2 x 2 tiles of 16)

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<float> {
  using acc_t = f32x4;
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
  static __device__ __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma<double> {
  using acc_t = f64x4;
  static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
  static __device__ __forceinline__ acc_t step(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// One slab: the 32 bands of each operand times kSlab grid points, stored
// [band][point] (rows padded by one element); each thread moves kVec
// consecutive complex elements (16 bytes) of each operand kLoads times.
template <typename T>
struct OvStage {
  using C = typename cx<T>::t;
  using V = typename std::conditional<sizeof(T) == 4, float4, double2>::type;  // 16 bytes
  static constexpr int kSlab = sizeof(T) == 4 ? 32 : 16;  // two slabs of both operands within 64 KiB of LDS
  static constexpr int kVec = 16 / static_cast<int>(sizeof(C));
  static constexpr int kPerBand = kSlab / kVec;
  static constexpr int kLoads = kBlk * kPerBand / (64 * kOvWaves);
  static_assert(kLoads >= 1 && kBlk * kPerBand % (64 * kOvWaves) == 0, "slab does not divide over the threads");
  static_assert(kOvChunkMax % kOvSub == 0 && kOvSub % kSlab == 0 && kOvChunkMin % kSlab == 0,
                "chunks and sub-chunks of whole slabs");
};

// The instances of one launch.  A plan of many small instances would otherwise
// take two launches of a few workgroups for each (twelve Gamma cells of 16 to
// 40 points: 160 us of the 770 of an apply), so up to kOvItems share both.
struct OvItem {
  const void* psi;
  const void* vx;
  void* vmat;
  double* part;
  long long bs, npts;
  double dv;
  int nbands, nk, nt, span, nchunks;
  unsigned blk1, red1;  // end of its workgroups in the product and in the reduction
};
// N: instances a launch has room for; one by itself, since a launch takes longer
// by its arguments' size (apply with E_x and M of 8^3 FP64, two k-points of 3
// bands: 36.7 us with 16, 35.2 with one).
constexpr int kOvItems = 16;
template <int N>
struct OvArgs {
  OvItem it[N];
  int n;
};

// Workgroups of a launch, in rows of at most 2^22: a dimension of a grid holds
// less than 2^32 threads, which 256 of them to a workgroup reach at 2^24 (one
// k-point of 14000 bands on 72^3).
constexpr unsigned kOvRow = 1u << 22;
constexpr unsigned ov_rows(unsigned total) { return (total + kOvRow - 1) / kOvRow; }
static_assert(ov_rows(1) == 1 && ov_rows(kOvRow) == 1 && ov_rows(kOvRow + 1) == 2 && ov_rows(1u << 31) < 65536 &&
                  static_cast<unsigned long long>(kOvRow) * 256 < (1ull << 32),
              "grids of the overlap");
inline dim3 ov_grid(unsigned total) { return dim3(total < kOvRow ? total : kOvRow, ov_rows(total)); }
__device__ __forceinline__ unsigned ov_wg() { return blockIdx.y * kOvRow + blockIdx.x; }

// The instance of workgroup b, and b's number within it.
template <unsigned OvItem::*END, int N>
__device__ __forceinline__ const OvItem& ov_item(const OvArgs<N>& a, unsigned& b) {
  if constexpr (N == 1) return a.it[0];
  int i = 0;
  while (i + 1 < a.n && b >= a.it[i].*END) ++i;
  if (i > 0) b -= a.it[i - 1].*END;
  return a.it[i];
}

// workgroups of an instance: (k, chunk, block_i * nbj + block_j), the last fastest; 256 threads
template <typename T, int N>
__global__ __launch_bounds__(64 * kOvWaves) void k_overlap_mfma(const OvArgs<N> args) {
  using C = typename cx<T>::t;
  unsigned wg = ov_wg();
  if (wg >= args.it[args.n - 1].blk1) return;  // past the last row's end
  const OvItem& in = ov_item<&OvItem::blk1, N>(args, wg);
  const C* __restrict__ psi = static_cast<const C*>(in.psi);
  const C* __restrict__ vx = static_cast<const C*>(in.vx);
  double* __restrict__ part = in.part;
  const int nbands = in.nbands, nt = in.nt, span = in.span;
  const long long bs = in.bs, npts = in.npts;
  using M = Mfma<T>;
  using S = OvStage<T>;
  using V = typename S::V;
  using acc_t = typename M::acc_t;
  constexpr int kSlab = S::kSlab;
  __shared__ C sa[2][kBlk][kSlab + 1];
  __shared__ C sb[2][kBlk][kSlab + 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int nbj = (nt + 1) / 2;
  const int kc = wg / (nbj * nbj), bij = wg - kc * (nbj * nbj);
  const int bi = bij / nbj, bj = bij - bi * nbj;
  const int k = kc / in.nchunks, chunk = kc - k * in.nchunks;
  const long long c0 = static_cast<long long>(chunk) * span;
  const long long c1 = c0 + span < npts ? c0 + span : npts;
  const size_t kb = static_cast<size_t>(k) * nbands;
  // this wave's tile (ti, tj) of the block, and whether it lies inside M
  const int ti = 2 * bi + (wave >> 1), tj = 2 * bj + (wave & 1);
  const bool live = ti < nt && tj < nt;
  // thread t moves, per operand and load q, band row r and points p0 .. p0 + kVec - 1 of the slab
  V ra[S::kLoads], rb[S::kLoads];
  auto load = [&](long long e0) {
#pragma unroll
    for (int q = 0; q < S::kLoads; ++q) {
      const int id = t + q * 64 * kOvWaves;
      const int r = id / S::kPerBand, p0 = (id - r * S::kPerBand) * S::kVec;
      const long long e = e0 + p0;
      const int ia = bi * kBlk + r, jb = bj * kBlk + r;
      const C* pa = psi + (kb + (ia < nbands ? ia : 0)) * bs + e;
      const C* pb = vx + (kb + (jb < nbands ? jb : 0)) * bs + e;
      V va = {}, vb = {};
      const bool whole = e + S::kVec <= c1;
      if (whole && ia < nbands && (reinterpret_cast<uintptr_t>(pa) & 15) == 0) {
        va = *reinterpret_cast<const V*>(pa);
      } else if (ia < nbands) {  // grid end or an odd band stride: element by element
        C* x = reinterpret_cast<C*>(&va);
#pragma unroll
        for (int u = 0; u < S::kVec; ++u) x[u] = e + u < c1 ? pa[u] : C{T(0), T(0)};
      }
      if (whole && jb < nbands && (reinterpret_cast<uintptr_t>(pb) & 15) == 0) {
        vb = *reinterpret_cast<const V*>(pb);
      } else if (jb < nbands) {
        C* x = reinterpret_cast<C*>(&vb);
#pragma unroll
        for (int u = 0; u < S::kVec; ++u) x[u] = e + u < c1 ? pb[u] : C{T(0), T(0)};
      }
      ra[q] = va;
      rb[q] = vb;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int q = 0; q < S::kLoads; ++q) {
      const int id = t + q * 64 * kOvWaves;
      const int r = id / S::kPerBand, p0 = (id - r * S::kPerBand) * S::kVec;
      const C* ea = reinterpret_cast<const C*>(&ra[q]);
      const C* eb = reinterpret_cast<const C*>(&rb[q]);
#pragma unroll
      for (int u = 0; u < S::kVec; ++u) {
        sa[buf][r][p0 + u] = ea[u];
        sb[buf][r][p0 + u] = eb[u];
      }
    }
  };
  acc_t re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
  double dre[4] = {0.0, 0.0, 0.0, 0.0}, dim[4] = {0.0, 0.0, 0.0, 0.0};  // FP64 sums of the sub-chunks
  const int ia = (wave >> 1) * 16 + (lane & 15), jb = (wave & 1) * 16 + (lane & 15), kk = lane >> 4;
  int buf = 0;
  load(c0);
  store(0);
  __syncthreads();
  for (long long e0 = c0; e0 < c1; e0 += kSlab) {
    const bool more = e0 + kSlab < c1;
    if (more) load(e0 + kSlab);  // the next slab's loads are in flight while this one is multiplied
    if (live) {
#pragma unroll
      for (int s4 = 0; s4 < kSlab; s4 += 4) {
        const C av = sa[buf][ia][s4 + kk];
        const C bv = sb[buf][jb][s4 + kk];
        re = M::step(av.x, bv.x, re);
        re = M::step(av.y, bv.y, re);
        im = M::step(av.x, bv.y, im);
        im = M::step(-av.y, bv.x, im);
      }
      if (!more || (e0 + kSlab - c0) % kOvSub == 0) {  // end of a sub-chunk: fold into FP64
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          dre[v] += static_cast<double>(re[v]);
          dim[v] += static_cast<double>(im[v]);
        }
        re = acc_t{0, 0, 0, 0};
        im = acc_t{0, 0, 0, 0};
      }
    }
    if (more) store(buf ^ 1);  // that buffer was last read before the previous barrier
    __syncthreads();
    buf ^= 1;
  }
  if (!live) return;
  double* dst = part + ((static_cast<size_t>(chunk) * in.nk + k) * (static_cast<size_t>(nt) * nt) +
                        static_cast<size_t>(ti) * nt + tj) * 512;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = M::row(lane, v), col = lane & 15;
    dst[(row * 16 + col) * 2] = dre[v];
    dst[(row * 16 + col) * 2 + 1] = dim[v];
  }
}

// vmat[k][i][j] = dV sum_chunks part[chunk][k][tile][row][col].  One workgroup
// per (k, tile, row): 16 columns x 16 shares of the chunks, each share summed
// in order, then the shares in order (one thread per element over all chunks
// waits on one load after another: at a Gamma cell of 48 bands that chain is
// longer than the product itself).
template <typename T, int N>
__global__ __launch_bounds__(256) void k_overlap_reduce(const OvArgs<N> args) {
  using C = typename cx<T>::t;
  __shared__ double2 red[16][16];
  unsigned wg = ov_wg();
  if (wg >= args.it[args.n - 1].red1) return;
  const OvItem& in = ov_item<&OvItem::red1, N>(args, wg);
  const double2* __restrict__ part = reinterpret_cast<const double2*>(in.part);
  C* __restrict__ vmat = static_cast<C*>(in.vmat);
  const int nbands = in.nbands, nchunks = in.nchunks, nk = in.nk, ntj = in.nt, tiles = in.nt * in.nt;
  const double dv = in.dv;
  const int k = wg / (tiles * 16), kt = wg - k * (tiles * 16);
  const int row = kt & 15, tile = kt >> 4;
  const int ti = tile / ntj, tj = tile - ti * ntj;
  const int i = ti * 16 + row;
  if (i >= nbands) return;  // the whole workgroup
  const int col = threadIdx.x & 15, share = threadIdx.x >> 4;
  const size_t step = static_cast<size_t>(nk) * tiles * 256;  // elements from chunk to chunk
  const double2* src = part + (static_cast<size_t>(k) * tiles + tile) * 256 + row * 16 + col;
  double sr = 0.0, si = 0.0;
#pragma unroll 4
  for (int c = share; c < nchunks; c += 16) {
    const double2 v = src[c * step];
    sr += v.x;
    si += v.y;
  }
  red[share][col] = double2{sr, si};
  __syncthreads();
  const int j = tj * 16 + col;
  if (share != 0 || j >= nbands) return;
#pragma unroll
  for (int s = 1; s < 16; ++s) {
    sr += red[s][col].x;
    si += red[s][col].y;
  }
  vmat[(static_cast<size_t>(k) * nbands + i) * nbands + j] = C{static_cast<T>(sr * dv), static_cast<T>(si * dv)};
}

template <typename T>
hipError_t launch_items(const Plan& p, const OvArgs<kOvItems>& a) {
  const OvItem& last = a.it[a.n - 1];
  p.prof.begin(FOCK_K_OVERLAP, p.stream);
  if (a.n == 1) {
    const OvArgs<1> one{{a.it[0]}, 1};
    hipLaunchKernelGGL((k_overlap_mfma<T, 1>), ov_grid(last.blk1), dim3(64 * kOvWaves), 0, p.stream, one);
    hipLaunchKernelGGL((k_overlap_reduce<T, 1>), ov_grid(last.red1), dim3(256), 0, p.stream, one);
  } else {
    hipLaunchKernelGGL((k_overlap_mfma<T, kOvItems>), ov_grid(last.blk1), dim3(64 * kOvWaves), 0, p.stream, a);
    hipLaunchKernelGGL((k_overlap_reduce<T, kOvItems>), ov_grid(last.red1), dim3(256), 0, p.stream, a);
  }
  p.prof.end(FOCK_K_OVERLAP, p.stream);
  return hipGetLastError();
}

template <typename T>
hipError_t overlaps_t(const Plan& p, const void* const* psi, void* const* vx, void* const* vmat) {
  const size_t room = std::max(p.tbuf_bytes, p.ovl_bytes);  // the pair buffer's memory, free by now
  OvArgs<kOvItems> a{};
  size_t used = 0;
  for (size_t i = 0; i < p.inst.size(); ++i) {
    if (!vmat[i]) continue;
    const Instance& in = p.inst[i];
    const size_t bytes = overlap_scratch_bytes(in, in.ovl_span);
    if (a.n == kOvItems || (a.n > 0 && used + bytes > room)) {
      const hipError_t e = launch_items<T>(p, a);
      if (e != hipSuccess) return e;
      a.n = 0;
      used = 0;
    }
    const unsigned blk0 = a.n ? a.it[a.n - 1].blk1 : 0, red0 = a.n ? a.it[a.n - 1].red1 : 0;
    OvItem& t = a.it[a.n++];
    t.psi = psi[i];
    t.vx = vx[i];
    t.vmat = vmat[i];
    t.part = reinterpret_cast<double*>(p.ws + p.ovl_off + used);
    t.bs = static_cast<long long>(in.band_stride);
    t.npts = static_cast<long long>(in.npts);
    t.dv = in.omega / static_cast<double>(in.npts);
    t.nbands = in.nbands;
    t.nk = in.nk;
    t.nt = (in.nbands + 15) / 16;
    t.span = in.ovl_span;
    t.nchunks = static_cast<int>((in.npts + t.span - 1) / t.span);
    const unsigned nbj = (t.nt + 1) / 2;
    t.blk1 = blk0 + nbj * nbj * t.nchunks * t.nk;
    t.red1 = red0 + static_cast<unsigned>(t.nt) * t.nt * 16 * t.nk;
    used += bytes;
  }
  return a.n ? launch_items<T>(p, a) : hipSuccess;
}

}  // namespace

// Grid points per workgroup (split-K chunk).  A workgroup waits out one slab
// load after another, about 1 us a slab, so a chunk of 4096 points takes about
// 130 (FP32) to 250 us (FP64) however small the problem is.  The chunks are
// made short enough for about 1024 workgroups (four per compute unit, what LDS
// holds), as long as the grid has them, and stay at 4096 points where that
// many are there anyway.  One apply with its overlap, always 4096 points
// against this rule: 16^3 Gamma, 8 bands, FP64 285 -> 36 us; 48^3 Gamma, 48
// bands, mixed 3.19 -> 2.93 ms; 32^3 2x2x2, 18 bands, FP64 (with the gradient)
// 12.79 -> 12.40 ms; 72^3 2x2x2, 24 bands, FP32 77.0 ms both ways.
// On small grids the shortest chunk is a 128th of the grid, down to 32 points:
// 12x10x9 FP64, two k-points of three bands, 12.9 -> 5.3 us (9 chunks -> 34).
int overlap_span(const Instance& in) {
  const long long nbj = ((in.nbands + 15) / 16 + 1) / 2;
  const long long want = std::max<long long>(1, 1024 / (nbj * nbj * in.nk));  // chunks
  const long long least = std::max<long long>(kOvChunkMin, std::min<long long>(128, in.npts / 128));
  const long long span = std::max(least, (in.npts + want - 1) / want);
  return static_cast<int>(std::min<long long>(kOvChunkMax, (span + kOvChunkMin - 1) / kOvChunkMin * kOvChunkMin));
}

size_t overlap_scratch_bytes(const Instance& in, int span) {
  const size_t nt = (in.nbands + 15) / 16;
  const size_t nchunks = (in.npts + span - 1) / span;
  return nchunks * in.nk * nt * nt * 512 * sizeof(double);
}

hipError_t launch_overlaps(const Plan& p, const void* const* psi, void* const* vx, void* const* vmat) {
  return p.io64() ? overlaps_t<double>(p, psi, vx, vmat) : overlaps_t<float>(p, psi, vx, vmat);
}

}  // namespace fock
