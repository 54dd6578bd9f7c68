// Device buffers of one context and the launch entry points of the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "coef.hpp"

namespace ddcc {

// MODE_STREAM is MODE_STEP with nontemporal stores of everything the step
// writes; the host picks it for grids whose step does not fit the 256 MB
// memory-side cache (there it is 3-6 % faster; on cache-resident grids
// plain stores are, by up to 19 %).
// MODE_RAGGED (2D) is MODE_STREAM without nontemporal accesses, for grids
// whose rows do not start on cache lines: a line there is written by two
// wavefronts, and only the caches can join the two parts (us per step, same
// GPU, nontemporal -> plain: 1500 x 1333 N = 2 FP32 193 -> 159, 1501 x 1333 N =
// 3 FP32 275 -> 219, 2050 x 2048 N = 3 FP32 580 -> 471, 1500 x 1333 N = 2 FP64
// 295 either way).
// MODE_FORK (2D, FP64 and FP32) is MODE_STEP with the history read from
// Bufs::histA, for steps from one stored state to another.
enum {
  MODE_STEP = 0,
  MODE_INIT = 1,
  MODE_MOMENTS = 2,
  MODE_STREAM = 3,
  MODE_FORK = 4,
  MODE_RAGGED = 5
};

// Pointers handed to the step/init/moments kernels (by value).
//   fA/gA/TA: current level (read), fB/gB/TB: next level (written);
//   in MODE_INIT the kernels write fB/gB/TB and read inC/inU/inP;
//   in MODE_MOMENTS they write outC/outU/outP and nothing else.
// Pop is the storage type of the moving populations (f^i_p, p >= 1, and
// g_p); S that of the history, T and geometry fields.
template <class Pop, class S>
struct Bufs {
  const Pop* fA;   // moving phase populations [N][Q-1][n] (phase_plane)
  Pop* fB;
  const double* f0A;  // rest populations of the phase sets [N][n], float64
  double* f0B;
  const Pop* gA;
  Pop* gB;
  S* hist;
  const S* histA;  // MODE_FORK: the history read
  const S* TA;
  S* TB;
  const S* psi;
  // wetting weights E_i = sum_k cos theta^k_iN |grad psi_k| over the walls,
  // [N-1][n] (eqs. 2.9, 2.14; Section 4.5)
  const S* wet;
  const double* inC;
  const double* inU;
  const double* inP;
  // moments: plane i of C at outC + i * out_n, of u likewise (2D; the 3D
  // planes of in* and out* are dense, nx ny nz nodes)
  double* outC;
  double* outU;
  double* outP;
  long long out_n;
  double* fC;      // 3D work fields: C_i [N][n] and mu_i [N][n], float64
  double* fmu;
  // device copies of the context's coefficients, Coef<double> and Coef<S>
  // (read by scalar loads instead of kernel arguments: the single-context
  // 2D kernel, and the 3D step kernel for some storage types)
  const void* coef_d;
  const void* coef_r;
};

// A population value v written in a narrower storage type: returns the
// stored value and adds the rounding v - stored to comp, so that the float64
// rest population can take it back and the phase mass stays exact.
template <class Pop, class R>
__device__ inline Pop narrow(R v, double& comp) {
  const Pop s = Pop(v);
  if constexpr (sizeof(Pop) < sizeof(R)) comp += double(v) - double(R(s));
  return s;
}

// kd: the float64 constants (fields C, mu, psi, rest populations);
// k: the same constants in the collision arithmetic type R; cus: compute
// units of the device.
template <class Pop, class S, class R>
hipError_t launch_2d(int nphase, int mode, const Coef<double>& kd,
                     const Coef<R>& k, const Bufs<Pop, S>& b, int ty, int cus,
                     hipStream_t st);

// Default tile height of launch_2d for a box; pop_bytes: size of the population
// type.
int default_tile_2d(int nx, int ny, int nphase, size_t pop_bytes, int cus);

// lattice_f: the phase-set lattice id (D3Q15 or D3Q7 of lattice.hpp); cus:
// compute units of the device.
template <class Pop, class S, class R>
hipError_t launch_3d(int nphase, int lattice_f, int mode,
                     const Coef<double>& kd, const Coef<R>& k,
                     const Bufs<Pop, S>& b, int tx, int ty, int cus,
                     hipStream_t st);

// Batches of independent 2D boxes: one list entry per tile, and the
// size and node offset of every instance. Each plane of each buffer holds
// every instance, instance i at nodes [off_i, off_i + n_i); the plane stride
// is the total node count (the n of the Coef handed to the batch kernel).
struct BatchTile {
  int inst, x0, y0, pad;
};
struct BatchInst {
  int nx, ny;
  long long n, off;
};

// One step (or initialisation, or moment read-out) of the ntiles >= 1 tiles
// listed, one workgroup each. kd, k: device tables of the coefficients of
// every instance.
template <class Pop, class S, class R>
hipError_t launch_2d_batch(int nphase, int mode, const Coef<double>* kd,
                           const Coef<R>* k, const Bufs<Pop, S>& b,
                           const BatchTile* tiles, const BatchInst* insts,
                           unsigned ntiles, int ty, hipStream_t st);

// Geometry from K walls: psi = prod_k psi_k and the wetting weights
// E_i = sum_k cos theta^k_iN |grad psi_k| (i < N-1), the gradient by the
// fixed isotropic stencil (D2Q9 at nz = 1, else D3Q19) on the periodic
// nx x ny x nz box. Inputs float64 on the device: psik [K][n], ctk
// [K][N-1][n] (NULL: 90 degrees). Outputs in S from node off on in planes of
// plane_stride nodes with rows px apart.
template <class S>
hipError_t launch_wet_field(const double* psik, const double* ctk, int K,
                            int nm1, int nx, int ny, int nz, int px,
                            S* psi_out, S* wet_out, long long plane_stride,
                            long long off, hipStream_t st);

// Copy rows of nx elements of esz (2, 4 or 8) bytes, px apart at `padded`, to
// dense rows at `dense` (pack) or from them.
hipError_t launch_copy_rows(void* padded, void* dense, bool pack, int nx,
                            int px, long long rows, size_t esz, hipStream_t st);

// Per-phase sums of all populations (rest plane f0 [N][stride_n] plus
// the moving planes of f [N][Q-1][stride_n], nodes [0, n) of each plane) into
// partial[block * N + i], plus a non-finite flag per block in bad[block] (if
// not NULL). first (may be NULL): *first = t if any population was not finite
// and *first is -1.
template <class Pop>
hipError_t launch_mass(const double* f0, const Pop* f, int nphase, int Q,
                       long long n, long long stride_n, double* partial,
                       int* bad, int nblocks, hipStream_t st,
                       long long* first = nullptr, long long t = 0);

// Blocks of the mass kernel whose partials fit the static workspace of the
// allocation-free mass check (the library never launches more).
constexpr int kScratchBlocks = 1024;

// Device address and size of that workspace on `device` (looked up once per
// device, with the device made current for the lookup).
hipError_t scratch_address(int device, void** ptr, size_t* bytes);

// out[i] = sum over blocks b in order of partial[b * N + i] (i < N, float64,
// as ddcc_mass sums them on the host); *nonfinite = OR of bad[0 .. nb) when
// nonfinite is not NULL. One workgroup.
hipError_t launch_mass_finish(const double* partial, const int* bad, int nb,
                              int N, double* out, int* nonfinite,
                              hipStream_t st);

// dst[i] = S(src[i]) for i < count.
template <class S>
hipError_t launch_convert(const double* src, S* dst, long long count,
                          hipStream_t st);

}  // namespace ddcc
