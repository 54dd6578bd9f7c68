// Reductions and conversions used by the host API.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace ddcc {

// Workspace of the mass check that allocates nothing (ddcc_mass_noalloc):
// the per-block partial sums [kScratchBlocks][kMaxN] float64, then the
// per-block non-finite flags [kScratchBlocks] int. One copy per GPU, held
// until the process ends; every call on a GPU shares it (calls that overlap
// on one GPU race). Host code never passes this name to a kernel: it takes
// the device address from scratch_address().
static __device__ __align__(256) unsigned char
    scratch[kScratchBlocks * kMaxN * sizeof(double) +
            kScratchBlocks * sizeof(int)];

namespace {

constexpr int kMassThreads = 256;
constexpr int kWaves = kMassThreads / 64;

// Per-phase population sums in float64: every thread accumulates a strided
// slice, wavefronts reduce with cross-lane shuffles, the four waves of the
// block through LDS; one partial per block and phase (summed in block order
// by the host or k_mass_finish, so the result is deterministic). bad (may be
// NULL): a non-finite flag per block; first (may be NULL): *first = t if a
// population was not finite and *first is still -1 (the time level of the
// first check that saw one). Bound by memory: N and Q are template
// parameters so that a node's N Q loads are in flight together (512^2 N = 3
// FP32: 12.4 us, and 4.6 us for a kernel of its own that gathered the flags,
// -> 7.7 us; with run-time loops each load waited for the one before).
template <int N, int Q, class S>
__global__ __launch_bounds__(kMassThreads) void k_mass(
    const double* __restrict__ f0, const S* __restrict__ f, long long n,
    long long stride_n, double* __restrict__ partial, int* __restrict__ bad,
    unsigned long long* first, long long t) {
  double acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = 0.0;
  int nonfinite = 0;
  const long long stride = (long long)gridDim.x * kMassThreads;
  for (long long x = (long long)blockIdx.x * kMassThreads + threadIdx.x; x < n;
       x += stride) {
    double s[N];
    S v[N][Q - 1];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      s[i] = f0[(long long)i * stride_n + x];
#pragma unroll
      for (int p = 1; p < Q; ++p) v[i][p - 1] = phase_plane(f, i, p, Q, stride_n)[x];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int p = 1; p < Q; ++p) s[i] += double(v[i][p - 1]);
      if (!isfinite(s[i])) nonfinite = 1;
      acc[i] += s[i];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    for (int off = 32; off > 0; off >>= 1) acc[i] += __shfl_xor(acc[i], off);
  for (int off = 32; off > 0; off >>= 1) nonfinite |= __shfl_xor(nonfinite, off);
  __shared__ double red[kWaves][N];
  __shared__ int redbad[kWaves];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) red[wave][i] = acc[i];
    redbad[wave] = nonfinite;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int b = 0;
    for (int w = 0; w < kWaves; ++w) b |= redbad[w];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      double s = 0.0;
      for (int w = 0; w < kWaves; ++w) s += red[w][i];
      partial[(long long)blockIdx.x * N + i] = s;
    }
    if (bad) bad[blockIdx.x] = b;
    if (b && first) atomicCAS(first, ~0ull, (unsigned long long)t);
  }
}

template <class S>
__global__ void k_convert(const double* src, S* dst, long long count) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
       i < count; i += stride)
    dst[i] = S(src[i]);
}

// Rows of nx elements px apart at `padded` to or from dense rows. One element
// per thread.
template <class E, bool PACK>
__global__ void k_copy_rows(E* padded, E* dense, int nx, int px,
                            long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const long long row = i / nx;
  const long long o = row * px + (i - row * nx);
  if constexpr (PACK)
    dense[i] = padded[o];
  else
    padded[o] = dense[i];
}

// Wetting weights of K walls (see launch_wet_field). One node per thread.
template <class S>
__global__ void k_wet_field(const double* psik, const double* ctk, int K,
                            int nm1, int nx, int ny, int nz, int px,
                            S* psi_out, S* wet_out, long long stride,
                            long long off) {
  const long long n = (long long)nx * ny * nz;
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n) return;
  const int x = int(idx % nx);
  const int y = int((idx / nx) % ny);
  const int z = int(idx / ((long long)nx * ny));
  double ps = 1.0;
  double E[kMaxN - 1] = {0.0, 0.0, 0.0};
  for (int kk = 0; kk < K; ++kk) {
    const double* p = psik + kk * n;
    ps *= p[idx];
    double g[3] = {0.0, 0.0, 0.0};
    // isotropic stencil: D2Q9 (1/3 axes, 1/12 diagonals) or D3Q19 (1/6
    // faces, 1/12 edges) weights at d0 = 1/3 over c_s^2 = 1/3
    for (int dz = (nz > 1 ? -1 : 0); dz <= (nz > 1 ? 1 : 0); ++dz)
      for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
          const int m = dx * dx + dy * dy + dz * dz;
          if (m == 0 || (nz > 1 && m == 3)) continue;
          const double w = nz > 1 ? (m == 1 ? 1.0 / 6.0 : 1.0 / 12.0)
                                  : (m == 1 ? 1.0 / 3.0 : 1.0 / 12.0);
          const int xs = (x + dx + nx) % nx, ys = (y + dy + ny) % ny;
          const int zs = nz > 1 ? (z + dz + nz) % nz : 0;
          const double v = p[((long long)zs * ny + ys) * nx + xs];
          g[0] += w * dx * v;
          g[1] += w * dy * v;
          g[2] += w * dz * v;
        }
    const double ag = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
    for (int i = 0; i < nm1; ++i) {
      const double c = ctk ? ctk[((long long)kk * nm1 + i) * n + idx] : 0.0;
      E[i] += c * ag;
    }
  }
  const long long o = off + ((long long)z * ny + y) * px + x;
  psi_out[o] = S(ps);
  for (int i = 0; i < nm1; ++i) wet_out[i * stride + o] = S(E[i]);
}

// Per-phase totals from the per-block partials, summed in block order by
// one lane per phase (the order and arithmetic of ddcc_mass's host sum, so
// the two agree bit for bit), and the OR of the block flags. The order makes
// a chain of nb additions; the partials are staged in LDS so that the chain
// waits for additions alone (1024 blocks, N = 3: 104 -> 17 us).
constexpr int kFinishThreads = 256;
__global__ __launch_bounds__(kFinishThreads) void k_mass_finish(
    const double* __restrict__ partial, const int* __restrict__ bad, int nb,
    int N, double* out, int* nonfinite) {
  __shared__ double part[kScratchBlocks * kMaxN];
  __shared__ int flag[kFinishThreads / 64];
  for (int q = threadIdx.x; q < nb * N; q += kFinishThreads) part[q] = partial[q];
  int f = 0;
  if (nonfinite)
    for (int b = threadIdx.x; b < nb; b += kFinishThreads) f |= bad[b];
  for (int off = 32; off > 0; off >>= 1) f |= __shfl_xor(f, off);
  if (threadIdx.x % 64 == 0) flag[threadIdx.x / 64] = f;
  __syncthreads();
  const int i = int(threadIdx.x);
  if (i < N) {
    double s = 0.0;
    int b = 0;
    for (; b + 32 <= nb; b += 32) {  // 32 LDS reads in flight, then 32 adds
      double v[32];
#pragma unroll
      for (int q = 0; q < 32; ++q) v[q] = part[(b + q) * N + i];
#pragma unroll
      for (int q = 0; q < 32; ++q) s += v[q];
    }
    for (; b < nb; ++b) s += part[b * N + i];
    out[i] = s;
  }
  if (nonfinite && i == 0) {
    int any = 0;
    for (int w = 0; w < kFinishThreads / 64; ++w) any |= flag[w];
    *nonfinite = any;
  }
}

}  // namespace

hipError_t scratch_address(int device, void** ptr, size_t* bytes) {
  // Device addresses of `scratch`, looked up once per device with that
  // device current (each GPU holds its own copy at its own address).
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  *ptr = nullptr;
  *bytes = sizeof(scratch);
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    int prev = -1;
    hipError_t e = hipGetDevice(&prev);
    if (e != hipSuccess) return e;
    if (prev != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (prev != device) {
      const hipError_t e2 = hipSetDevice(prev);
      if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return e;
    addr[device] = p;
  }
  *ptr = addr[device];
  return hipSuccess;
}

hipError_t launch_mass_finish(const double* partial, const int* bad, int nb,
                              int N, double* out, int* nonfinite,
                              hipStream_t st) {
  if (nb < 1 || nb > kScratchBlocks || N < 1 || N > kMaxN || !out ||
      (nonfinite && !bad))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mass_finish, dim3(1), dim3(kFinishThreads), 0, st, partial, bad,
                     nb, N, out, nonfinite);
  return hipGetLastError();
}

namespace {
template <class E>
hipError_t copy_rows_as(void* padded, void* dense, bool pack, int nx, int px,
                        long long count, hipStream_t st) {
  const dim3 grid((unsigned)((count + 255) / 256));
  E* a = static_cast<E*>(padded);
  E* b = static_cast<E*>(dense);
  if (pack)
    hipLaunchKernelGGL((k_copy_rows<E, true>), grid, dim3(256), 0, st, a, b, nx,
                       px, count);
  else
    hipLaunchKernelGGL((k_copy_rows<E, false>), grid, dim3(256), 0, st, a, b,
                       nx, px, count);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_copy_rows(void* padded, void* dense, bool pack, int nx,
                            int px, long long rows, size_t esz,
                            hipStream_t st) {
  const long long count = rows * nx;
  if (nx < 1 || px < nx || rows < 1 || (count + 255) / 256 > 0x7fffffffLL)
    return hipErrorInvalidValue;
  if (esz == 8)
    return copy_rows_as<uint64_t>(padded, dense, pack, nx, px, count, st);
  if (esz == 4)
    return copy_rows_as<uint32_t>(padded, dense, pack, nx, px, count, st);
  if (esz == 2)
    return copy_rows_as<uint16_t>(padded, dense, pack, nx, px, count, st);
  return hipErrorInvalidValue;
}

template <class S>
hipError_t launch_wet_field(const double* psik, const double* ctk, int K,
                            int nm1, int nx, int ny, int nz, int px,
                            S* psi_out, S* wet_out, long long plane_stride,
                            long long off, hipStream_t st) {
  const long long n = (long long)nx * ny * nz;
  if (n <= 0 || px < nx || K < 1 || nm1 < 0 || nm1 > kMaxN - 1)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_wet_field<S>), dim3((unsigned)((n + 255) / 256)),
                     dim3(256), 0, st, psik, ctk, K, nm1, nx, ny, nz, px,
                     psi_out, wet_out, plane_stride, off);
  return hipGetLastError();
}

template hipError_t launch_wet_field<double>(const double*, const double*, int,
                                             int, int, int, int, int, double*,
                                             double*, long long, long long,
                                             hipStream_t);
template hipError_t launch_wet_field<float>(const double*, const double*, int,
                                            int, int, int, int, int, float*,
                                            float*, long long, long long,
                                            hipStream_t);

template <class S>
hipError_t launch_mass(const double* f0, const S* f, int nphase, int Q,
                       long long n, long long stride_n, double* partial,
                       int* bad, int nblocks, hipStream_t st, long long* first,
                       long long t) {
  auto go = [&](auto nc, auto qc) {
    constexpr int N = decltype(nc)::value, QC = decltype(qc)::value;
    hipLaunchKernelGGL((k_mass<N, QC, S>), dim3(nblocks), dim3(kMassThreads),
                       0, st, f0, f, n, stride_n, partial, bad,
                       reinterpret_cast<unsigned long long*>(first), t);
    return hipGetLastError();
  };
  using std::integral_constant;
  const integral_constant<int, 2> n2{};
  const integral_constant<int, 3> n3{};
  switch (Q) {
    case 9: {
      const auto q = integral_constant<int, 9>();
      if (nphase == 2) return go(n2, q);
      if (nphase == 3) return go(n3, q);
      if (nphase == 4) return go(integral_constant<int, 4>(), q);
      break;
    }
    case 7: {
      const auto q = integral_constant<int, 7>();
      if (nphase == 2) return go(n2, q);
      if (nphase == 3) return go(n3, q);
      break;
    }
    case 15: {
      const auto q = integral_constant<int, 15>();
      if (nphase == 2) return go(n2, q);
      if (nphase == 3) return go(n3, q);
      break;
    }
  }
  return hipErrorInvalidValue;
}

template <class S>
hipError_t launch_convert(const double* src, S* dst, long long count,
                          hipStream_t st) {
  if (count <= 0) return hipSuccess;
  long long blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL((k_convert<S>), dim3((unsigned)blocks), dim3(256), 0, st,
                     src, dst, count);
  return hipGetLastError();
}

template hipError_t launch_mass<double>(const double*, const double*, int, int,
                                         long long, long long, double*, int*,
                                         int, hipStream_t, long long*,
                                         long long);
template hipError_t launch_mass<float>(const double*, const float*, int, int,
                                         long long, long long, double*, int*,
                                         int, hipStream_t, long long*,
                                         long long);
template hipError_t launch_mass<_Float16>(const double*, const _Float16*, int, int,
                                         long long, long long, double*, int*,
                                         int, hipStream_t, long long*,
                                         long long);
template hipError_t launch_mass<__bf16>(const double*, const __bf16*, int, int,
                                         long long, long long, double*, int*,
                                         int, hipStream_t, long long*,
                                         long long);
template hipError_t launch_convert<double>(const double*, double*, long long,
                                           hipStream_t);
template hipError_t launch_convert<float>(const double*, float*, long long,
                                          hipStream_t);

}  // namespace ddcc
