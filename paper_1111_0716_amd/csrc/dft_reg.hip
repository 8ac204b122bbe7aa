// Register-line kernels of the batched 3-D DFT (fock_dft3) on grids N1 x L x L:
// every 1-D transform runs in one lane's registers on a whole line
// (reg_fft.hpp), a plane switches axes through a padded LDS transpose.  One
// barrier chain shorter than the tiles of pass_line.hip, which counts on small
// grids where a call is short (256 DFTs of 16^3 FP32 10 against 15.5 us, 75 of
// 24^3 13.8 against 16.7) and up to 48 points in FP32 where the caches hold the
// data (reg_dft_use); large batches are bound by memory on both.
#include <algorithm>

#include "fft_lds.hpp"
#include "fock_internal.hpp"
#include "pass_common.hpp"
#include "reg_fft.hpp"

namespace fock {

template <typename T, int L>
struct DftShape {
  static constexpr int LP = L + 1;  // padded LDS row
  // axis switches go through LDS one component (real, then imaginary) at a time
  static constexpr int PLANE_LDS = L * LP * static_cast<int>(sizeof(T));
  static constexpr int PL = 256 / L;  // planes per workgroup
  static constexpr int NTP = PL * L;  // threads of the plane pass
  static constexpr int LDS = PL * PLANE_LDS;
};

// Switch a plane's axis: thread `col` holds line x[i] = P[i][col]; afterwards
// it holds x[i] = P[col][i].  One component at a time through sp ([L][LP]
// of T, this plane's share of LDS); every thread of the block must call it.
template <typename C, typename T, int L>
__device__ __forceinline__ void transpose_plane(C* x, T* sp, int col) {
  constexpr int LP = L + 1;
  __syncthreads();  // earlier readers of sp are done
#pragma unroll
  for (int i = 0; i < L; ++i) sp[i * LP + col] = x[i].x;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < L; ++i) x[i].x = sp[col * LP + i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < L; ++i) sp[i * LP + col] = x[i].y;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < L; ++i) x[i].y = sp[col * LP + i];
}

// plane pass: axes 2 and 3 of plane j1, read and written as columns (one
// line per lane, coalesced); two transposes bring the rows in and back out
template <typename T, int L, int S>
__global__ __launch_bounds__((DftShape<T, L>::NTP), 2) void k_dft_plane_reg(
    int n1, typename cx<T>::t* __restrict__ data, long long stride) {
  using C = typename cx<T>::t;
  using Sh = DftShape<T, L>;
  constexpr int LL = L * L;
  extern __shared__ unsigned char smem_raw[];
  const int t = threadIdx.x, pl = t / L, col = t - (t / L) * L;
  const int j1 = blockIdx.x * Sh::PL + pl;
  const bool valid = j1 < n1;
  T* sp = reinterpret_cast<T*>(smem_raw) + pl * L * Sh::LP;
  C* g = data + static_cast<size_t>(blockIdx.y) * stride + static_cast<size_t>(j1) * LL + col;
  C x[L];
#pragma unroll
  for (int j2 = 0; j2 < L; ++j2) x[j2] = valid ? g[j2 * L] : C{T(0), T(0)};
  reg_fft<C, L, S>(x);                  // axis 2: x[c2] at j3 = col
  transpose_plane<C, T, L>(x, sp, col);  // row c2 = col
  reg_fft<C, L, S>(x);                  // axis 3: x[c3]
  transpose_plane<C, T, L>(x, sp, col);  // column c3 = col: x[c2]
  if (valid) {
#pragma unroll
    for (int c2 = 0; c2 < L; ++c2) g[c2 * L] = x[c2];
  }
}

// pencil pass: axis 1 of line (c2, c3) = l, coalesced across lanes
template <typename T, int L, int S>
__global__ __launch_bounds__(256, 2) void k_dft_pencil_reg(
    int ll, typename cx<T>::t* __restrict__ data, long long stride) {
  using C = typename cx<T>::t;
  const int LL = ll;
  const int l = blockIdx.x * 256 + threadIdx.x;
  if (l >= LL) return;  // no barrier in this kernel
  C* g = data + static_cast<size_t>(blockIdx.y) * stride;
  const unsigned lo = static_cast<unsigned>(l) * sizeof(C);
  C x[L];
#pragma unroll
  for (int j1 = 0; j1 < L; ++j1) x[j1] = *lane_at(g + static_cast<size_t>(j1) * LL, lo);
  reg_fft<C, L, S>(x);
  const unsigned so = opaque(lo);
#pragma unroll
  for (int c1 = 0; c1 < L; ++c1) *lane_at(g + static_cast<size_t>(c1) * LL, so) = x[c1];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

template <typename T, int L, int S>
void dft_plane_L(const Plan& p, int n1, int count, typename cx<T>::t* d, long long stride) {
  using Sh = DftShape<T, L>;
  hipLaunchKernelGGL((k_dft_plane_reg<T, L, S>), dim3((n1 + Sh::PL - 1) / Sh::PL, count), dim3(Sh::NTP), Sh::LDS,
                     p.stream, n1, d, stride);
}

template <typename T, int L, int S>
void dft_pencil_L(const Plan& p, int ll, int count, typename cx<T>::t* d, long long stride) {
  hipLaunchKernelGGL((k_dft_pencil_reg<T, L, S>), dim3((ll + 255) / 256, count), dim3(256), 0, p.stream, ll, d,
                     stride);
}

// the lengths that run here (32 in FP64 and longer lines: pass_line.hip is as fast or faster)
#define FOCK_DFT_F32(X) X(16) X(24) X(32) X(36) X(40) X(48)
#define FOCK_DFT_F64(X) X(16) X(24)

// the lengths that run here at any size, and those that do at some
bool dft_len(fock_precision prec, int n) { return n == 16 || n == 24 || (n == 32 && prec == FOCK_C64); }
bool dft_len_cached(fock_precision prec, int n) {
  return dft_len(prec, n) || (prec == FOCK_C64 && (n == 36 || n == 40 || n == 48));
}

template <typename T, int S>
hipError_t reg_dft3_t(const Plan& p, int inst, int count, void* data, long long stride) {
  using C = typename cx<T>::t;
  const int* g = p.inst[inst].grid;
  C* d = static_cast<C*>(data);
  bool ok = false;
#define CASE(N) \
  case N: dft_plane_L<T, N, S>(p, g[0], count, d, stride); ok = true; break;
  if constexpr (sizeof(T) == 4) {
    switch (g[1]) { FOCK_DFT_F32(CASE) default: break; }
  } else {
    switch (g[1]) { FOCK_DFT_F64(CASE) default: break; }
  }
#undef CASE
  if (!ok) return hipErrorInvalidValue;
  ok = false;
#define CASE(N) \
  case N: dft_pencil_L<T, N, S>(p, g[1] * g[2], count, d, stride); ok = true; break;
  if constexpr (sizeof(T) == 4) {
    switch (g[0]) { FOCK_DFT_F32(CASE) default: break; }
  } else {
    switch (g[0]) { FOCK_DFT_F64(CASE) default: break; }
  }
#undef CASE
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

// FP32 lines of 36 to 48 points: where the batch fits the last-level cache but
// not the L2s.  Here / pass_line.hip, us: 36^3 FP32, 16 DFTs 16.6/15.8, 64 (24
// MB) 23.0/24.3, 128 31.4/35.5, 512 (191 MB) 99.9/103, 1024 (382 MB) 293/279;
// 40^3, 32 25.9/24.9, 64 (33 MB) 24.4/26.0; 48^3, 64 (57 MB) 36.4/38.3; 36x24x24,
// 256 (42 MB) 27.7/30.7.
bool reg_dft_use(fock_precision prec, const int grid[3], size_t bytes) {
  if (grid[1] != grid[2]) return false;
  if (dft_len(prec, grid[0]) && dft_len(prec, grid[1])) return true;
  return dft_len_cached(prec, grid[0]) && dft_len_cached(prec, grid[1]) && bytes > (size_t{20} << 20) &&
         bytes <= kLastLevelBytes;
}

hipError_t launch_reg_dft3(const Plan& p, int inst, int sign, int count, void* data, long long stride) {
  if (p.prec == FOCK_C64)
    return sign < 0 ? reg_dft3_t<float, -1>(p, inst, count, data, stride)
                    : reg_dft3_t<float, +1>(p, inst, count, data, stride);
  return sign < 0 ? reg_dft3_t<double, -1>(p, inst, count, data, stride)
                  : reg_dft3_t<double, +1>(p, inst, count, data, stride);
}

}  // namespace fock
