// The context behind the opaque ddcc_ctx handle of include/ddcc.h, shared by
// the host files of the library (not installed, not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "../../include/ddcc.h"
#include "coef.hpp"

using ddcc::Coef;

struct ddcc_ctx {
  ddcc_params p{};
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int device = 0;
  int cus = 0;  // compute units of the device
  long long n = 0;      // plane stride: px ny nz
  long long nodes = 0;  // nx ny nz
  int px = 0;           // row pitch of the planes (row_pitch; nx in 2D)
  int Qf = 0, Qg = 0, nhist = 0, nT = 0;
  size_t esz = 8;   // history, T and geometry fields
  size_t pesz = 8;  // moving populations
  void* f[2] = {nullptr, nullptr};
  double* f0[2] = {nullptr, nullptr};  // rest populations, float64
  void* g[2] = {nullptr, nullptr};
  void* T[2] = {nullptr, nullptr};
  void* hist = nullptr;
  void* psi = nullptr;
  void* wet = nullptr;         // wetting weights [N-1][n]
  double* work = nullptr;     // 3D: C_i and mu_i fields, 2 N n float64
  // 2D contexts with one wall: psi [n] and cos theta_iN [N-1][n] in
  // float64, for the adjoint's derivative of the wetting weights
  double* geo64 = nullptr;
  double* staging = nullptr;  // (N + dim + 1) * n float64, lazily
  double* partial = nullptr;
  int* bad = nullptr;
  int mass_blocks = 0;
  int cur = 0;
  bool geom_ok = false, fields_ok = false;
  int nwalls = 0;  // walls of the current geometry
  int64_t t = 0;
  int tile_x = 64, tile_y = 8;
  // steps run as MODE_STREAM (nontemporal stores): what one step moves does
  // not fit the memory-side cache
  bool stream_stores = false;
  // periodic in-stream diagnostics (ddcc_set_diagnostics)
  int diag_every = 0;
  int64_t diag_t = -1;          // time level of the last check
  double* diag_partial = nullptr;
  long long* diag_first = nullptr;  // first level that saw a non-finite value
  // second stream of the adjoint sweep and its events, made by the first
  // sweep and kept (making and destroying them took 0.4 ms per sweep)
  hipStream_t adj_stream = nullptr;
  hipEvent_t adj_events[5] = {};
  // Captured groups of steps of a small box (ddcc_step), by tile height (2, 4,
  // 8, 16), size and parity of cur, and the stream they are captured on.
  hipGraphExec_t step_graph[4][2][2] = {};
  hipStream_t capture_stream = nullptr;
  int64_t direct_steps = 0;    // steps launched one by one so far
  bool graphs_failed = false;  // a capture failed: no further attempt
  std::string err;
  Coef<double> kd{};
  Coef<float> kf{};
  Coef<double>* dkd = nullptr;  // device copies of kd and kf
  Coef<float>* dkf = nullptr;
};

namespace ddcc::detail {

// Record an error message on the context and return code.
int fail(ddcc_ctx* c, int code, const std::string& msg);
// Record a HIP error (DDCC_E_NOMEM for out-of-memory, else DDCC_E_HIP).
int hip_fail(ddcc_ctx* c, hipError_t e, const char* what);
// Makes a device current for its scope. Streams, events and graphs belong to
// the device that is current where they are made; those a context makes after
// ddcc_create have to be on its own.
class OnDevice {
 public:
  explicit OnDevice(int device) {
    status = hipGetDevice(&before_);
    if (status != hipSuccess || before_ == device) return;
    status = hipSetDevice(device);
    moved_ = status == hipSuccess;
  }
  ~OnDevice() {
    if (moved_) (void)hipSetDevice(before_);
  }
  OnDevice(const OnDevice&) = delete;
  OnDevice& operator=(const OnDevice&) = delete;
  hipError_t status;

 private:
  int before_ = 0;
  bool moved_ = false;
};

// Launch one forward step on the current buffers (the caller flips cur and
// advances t).
hipError_t step_launch(ddcc_ctx* c);

}  // namespace ddcc::detail
