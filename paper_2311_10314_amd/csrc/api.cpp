// Host side of the C ABI declared in include/ddcc.h: parameter validation,
// derived constants, device buffers (A-B population pairs), kernel launches.
#include <hip/hip_runtime.h>

#include <array>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/ddcc.h"
#include "coef.hpp"
#include "ctx.hpp"
#include "kernels.hpp"
#include "lattice.hpp"

using namespace ddcc;

namespace {

const char* kVersion = "ddcc 0.1 (gfx950)";

// Memory-side (Infinity) cache of the chip. A step that moves more than
// this streams its outputs (MODE_STREAM): 256^3 3D and 2048^2 2D steps 3-6 %
// faster; on a 512^2 box, whose step stays in this cache, plain stores are
// 19 % faster.
constexpr size_t kCacheBytes = size_t(256) << 20;

// Bytes one step moves: the populations (one buffer read, the other
// written), T likewise, the in-place history read and written, and the 3D
// work fields written and read.
size_t step_bytes(size_t pops, size_t T, size_t hist, size_t work) {
  return 2 * (pops + T + hist + work);
}

// Whether rows of nx populations start where nontemporal stores of a row's
// 64-node pieces fill what they touch: on 64 bytes, or on 32 in FP64 (us per
// step, nontemporal / plain: rows on 64 bytes, 2064 x 2048 N = 3 FP32 505 / 533;
// on 32, 2056 x 2048 N = 3 FP32 521 / 462, 1500 x 1333 N = 2 FP64 290 / 293; on
// less, MODE_RAGGED).
bool rows_on_lines(long long nx, size_t bytes) {
  return nx * bytes % (bytes == 8 ? 32 : 64) == 0;
}

int fail(ddcc_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

// The runtime keeps an error until it is read: reading it here keeps it out of
// the check of a later kernel launch.
int hip_fail(ddcc_ctx* c, hipError_t e, const char* what) {
  (void)hipGetLastError();
  std::string m = std::string(what) + ": " + hipGetErrorString(e);
  return fail(c, e == hipErrorOutOfMemory ? DDCC_E_NOMEM : DDCC_E_HIP, m);
}

#define HIPCHK(ctx, expr, what)                 \
  do {                                          \
    hipError_t e_ = (expr);                     \
    if (e_ != hipSuccess) return hip_fail(ctx, e_, what); \
  } while (0)

int lattice_q(int lat) {
  switch (lat) {
    case DDCC_D2Q9:
      return 9;
    case DDCC_D3Q7:
      return 7;
    case DDCC_D3Q15:
      return 15;
    case DDCC_D3Q19:
      return 19;
    default:
      return 0;
  }
}

// Weights w_p(d0) in the velocity order of lattice.hpp (Section 3 tables;
// D3Q19 from the same moment constraints). Returns false if any is <= 0.
bool lattice_weights(int lat, double d0, double* w) {
  double w0, w1, w2 = 0, w3 = 0;
  int q = lattice_q(lat);
  switch (lat) {
    case DDCC_D2Q9:
      w0 = (1 - d0) * (1 - d0);
      w1 = (d0 - d0 * d0) / 2;
      w2 = d0 * d0 / 4;
      for (int p = 0; p < 9; ++p) w[p] = p == 0 ? w0 : (p < 5 ? w1 : w2);
      break;
    case DDCC_D3Q7:
      w0 = 1 - 3 * d0;
      w1 = d0 / 2;
      for (int p = 0; p < 7; ++p) w[p] = p == 0 ? w0 : w1;
      break;
    case DDCC_D3Q15:
      w0 = 1 - 3 * d0 + 2 * d0 * d0;
      w1 = (d0 - d0 * d0) / 2;
      w3 = d0 * d0 / 8;
      for (int p = 0; p < 15; ++p) w[p] = p == 0 ? w0 : (p < 7 ? w1 : w3);
      break;
    case DDCC_D3Q19:
      w0 = 1 - 3 * d0 + 3 * d0 * d0;
      w1 = (d0 - 2 * d0 * d0) / 2;
      w2 = d0 * d0 / 4;
      for (int p = 0; p < 19; ++p) w[p] = p == 0 ? w0 : (p < 7 ? w1 : w2);
      break;
    default:
      return false;
  }
  for (int p = 0; p < q; ++p)
    if (!(w[p] > 0)) return false;
  return true;
}

bool finite(double x) { return std::isfinite(x); }

int validate(const ddcc_params* p, std::string& msg) {
  if (!p) {
    msg = "params is NULL";
    return DDCC_E_INVAL;
  }
  if (p->dim != 2 && p->dim != 3) {
    msg = "dim must be 2 or 3";
    return DDCC_E_INVAL;
  }
  if (p->nx < 1 || p->ny < 1 || p->nz < 1) {
    msg = "grid sizes must be >= 1";
    return DDCC_E_INVAL;
  }
  if (p->dim == 2 && p->nz != 1) {
    msg = "nz must be 1 in 2D";
    return DDCC_E_INVAL;
  }
  if ((long long)p->nx * p->ny * p->nz > (1LL << 29)) {
    msg = "grid larger than 2^29 nodes";
    return DDCC_E_INVAL;
  }
  if (p->nphase < 2 || p->nphase > DDCC_MAX_PHASES) {
    msg = "nphase must be in [2, 4]";
    return DDCC_E_INVAL;
  }
  if (p->precision != DDCC_FP64 && p->precision != DDCC_FP32 &&
      p->precision != DDCC_FP16 && p->precision != DDCC_BF16) {
    msg = "precision must be DDCC_FP64, DDCC_FP32, DDCC_FP16 or DDCC_BF16";
    return DDCC_E_INVAL;
  }
  if (p->dim == 2 && (p->lattice_f != DDCC_D2Q9 || p->lattice_g != DDCC_D2Q9)) {
    msg = "2D runs use D2Q9 for both sets";
    return DDCC_E_INVAL;
  }
  if (p->dim == 3 &&
      ((p->lattice_f != DDCC_D3Q15 && p->lattice_f != DDCC_D3Q7) ||
       (p->lattice_g != DDCC_D3Q19 && p->lattice_g != DDCC_D3Q15))) {
    msg = "3D runs use D3Q15/D3Q7 phase sets and a D3Q19/D3Q15 flow set";
    return DDCC_E_INVAL;
  }
  const double scal[] = {p->d0, p->eps, p->m0, p->rho0, p->psi_min, p->lam};
  for (double v : scal)
    if (!finite(v)) {
      msg = "non-finite scalar parameter";
      return DDCC_E_INVAL;
    }
  if (!(p->d0 > 0 && p->d0 < 1)) {
    msg = "d0 must be in (0, 1)";
    return DDCC_E_INVAL;
  }
  double w[19];
  if (!lattice_weights(p->lattice_f, p->d0, w) ||
      !lattice_weights(p->lattice_g, p->d0, w)) {
    msg = "d0 gives a non-positive lattice weight";
    return DDCC_E_INVAL;
  }
  if (!(p->eps > 0) || !(p->m0 > 0) || !(p->psi_min > 0) || !(p->lam >= 0)) {
    msg = "eps, m0, psi_min must be > 0 and lam >= 0";
    return DDCC_E_INVAL;
  }
  const int N = p->nphase;
  for (int i = 0; i < N; ++i) {
    if (!(p->rho[i] > 0) || !finite(p->rho[i]) || !(p->nu[i] > 0) ||
        !finite(p->nu[i]) || !finite(p->eta[i])) {
      msg = "rho_i and nu_i must be finite and > 0";
      return DDCC_E_INVAL;
    }
    for (int j = 0; j < N; ++j) {
      const double s = p->sigma[i][j];
      if (!finite(s) || s != p->sigma[j][i] || (i == j && s != 0) ||
          (i != j && !(s > 0))) {
        msg = "sigma must be symmetric, zero on the diagonal, > 0 elsewhere";
        return DDCC_E_INVAL;
      }
    }
  }
  for (int r = 0; r < 6; ++r) {
    if (!(p->s_f[r] > 0 && p->s_f[r] < 2)) {
      msg = "phase-set rates must be in (0, 2)";
      return DDCC_E_INVAL;
    }
    if ((r != DDCC_S21 && r != DDCC_S22) && !(p->s_g[r] > 0 && p->s_g[r] < 2)) {
      msg = "flow-set rates must be in (0, 2)";
      return DDCC_E_INVAL;
    }
  }
  for (int a = 0; a < 3; ++a)
    if (!finite(p->accel[a]) || !finite(p->force[a])) {
      msg = "non-finite body acceleration or force";
      return DDCC_E_INVAL;
    }
  return DDCC_OK;
}

template <class L>
void fourth_order_q_for(double d0, double q4[3][3]) {
  double w[19];
  lattice_weights(L::ID, d0, w);
  const double cs2 = d0;
  for (int j = 0; j < 3; ++j)
    for (int g = 0; g < 3; ++g) q4[j][g] = 0;
  for (int k = 0; k < L::Q; ++k) {
    const int j = g4_index<L>(k);
    if (j < 0) continue;
    for (int g = 0; g < L::D; ++g) {
      double s = 0;
      for (int p = 0; p < L::Q; ++p) {
        const int cg = g == 0 ? L::c[p].x : (g == 1 ? L::c[p].y : L::c[p].z);
        s += w[p] * row_value<L>(k, p, cs2) * (cg * cg - cs2);
      }
      s /= cs2 - cs2 * cs2;
      q4[j][g] = std::fabs(s) < 1e-14 ? 0.0 : s;
    }
  }
}

// q4 of coef.hpp for the flow lattice.
void fourth_order_q(int lat, double d0, double q4[3][3]) {
  switch (lat) {
    case DDCC_D3Q15:
      fourth_order_q_for<D3Q15>(d0, q4);
      break;
    case DDCC_D3Q19:
      fourth_order_q_for<D3Q19>(d0, q4);
      break;
    default:
      fourth_order_q_for<D2Q9>(d0, q4);
  }
}

int hist_planes(const ddcc_params& p) {
  // 2D: phi C_i u (2N), Y (3), P; 3D: phi C_i (N), u (3), m^C (3), P (1)
  return p.dim == 2 ? 2 * p.nphase + 4 : p.nphase + 7;
}

size_t pop_bytes(const ddcc_params& p) {
  return p.precision == DDCC_FP64 ? 8 : (p.precision == DDCC_FP32 ? 4 : 2);
}

size_t field_bytes(const ddcc_params& p) {
  return p.precision == DDCC_FP64 ? 8 : 4;
}

// step_bytes of a box whose planes hold n values.
size_t step_bytes_of(const ddcc_params& p, size_t n) {
  const size_t N = (size_t)p.nphase, d = (size_t)p.dim, e = field_bytes(p);
  return step_bytes((N * (lattice_q(p.lattice_f) - 1) + lattice_q(p.lattice_g)) *
                            n * pop_bytes(p) +
                        N * n * sizeof(double),
                    d * (d - 1) / 2 * n * e, hist_planes(p) * n * e,
                    d == 3 ? 2 * N * n * e : 0);
}

// Row pitch of the planes of a 3D box: rows padded to whole 128-byte lines of
// every array they are in (32 nodes; 16 in FP64). Otherwise the pieces of a row
// that wavefronts read and write start inside lines. us per step, rows as they
// are -> padded, one context / each of three at once, boxes of about 700000
// nodes: FP32 N = 2 75 nodes 193/174 -> 162/139, 100 162/155 -> 142/130, 130
// 186/174 -> 148/132; FP64 70 330/320 -> 272/244, 100 267/239 -> 256/224; FP16
// N = 3 130 238/228 -> 199/187. Not for rows that one tile spans (every line
// is in one workgroup's hands, and padding is only more lines: 33 nodes FP32
// 157/127 -> 175/155, 54 151/137 -> 148/144, 26 FP64 191/144 -> 204/178), nor
// where the padding is more than 30 % of a row, 25 in the 16-bit storages (100
// nodes FP16, 28 %, 107/101 -> 125/99). Boxes beyond 2^26 nodes, whose memory
// may be scarce, keep their rows too, and so do boxes whose step would leave the
// memory-side cache with its padding, or nearly (one context / each of three at
// once: 130 x 90 x 42 FP32 N = 2 119/104 -> 128/93, 110 x 110 x 37 86/82 ->
// 103/74, 80 x 110 x 36 N = 3, 0.97 of the cache with its padding, 77/86 ->
// 86/90, 80 x 110 x 79 FP16 118/107 -> 138/108; at 0.75 of the cache 150 x 100 x
// 25 FP32 84/77 -> 80/70).
int row_pitch(const ddcc_params& p) {
  if (p.dim != 3 || p.nx <= 64) return p.nx;
  const bool half = p.precision == DDCC_FP16 || p.precision == DDCC_BF16;
  const long long unit = p.precision == DDCC_FP64 ? 16 : 32;
  const long long px = (p.nx + unit - 1) / unit * unit;
  const long long most = (half ? 125 : 130) * (long long)p.nx / 100;
  if (px > most || px * p.ny * p.nz > (1LL << 26)) return p.nx;
  const size_t rows = (size_t)p.ny * p.nz;
  if (step_bytes_of(p, rows * p.nx) <= kCacheBytes &&
      step_bytes_of(p, rows * px) > kCacheBytes / 8 * 7)
    return p.nx;
  return (int)px;
}

template <class R>
void fill_coef(const ddcc_params& p, int px, long long n, Coef<R>& k) {
  std::memset(&k, 0, sizeof(k));
  const int N = p.nphase;
  const double cs2 = p.d0;
  k.nx = p.nx;
  k.ny = p.ny;
  k.nz = p.nz;
  k.px = px;
  k.n = n;
  k.cs2 = R(cs2);
  k.inv_cs2 = R(1.0 / cs2);
  k.psi_min = R(p.psi_min);
  k.lam = R(p.lam);
  k.rho0 = R(p.rho0);
  k.m0 = R(p.m0);
  for (int i = 0; i < N; ++i) {
    double eta = p.eta[i];
    if (!(eta > 0)) eta = p.m0 / ((1.0 / p.s_f[DDCC_S1] - 0.5) * cs2);  // eq. 17
    k.eta[i] = R(eta);
    k.rho[i] = R(p.rho[i]);
    k.nu[i] = R(p.nu[i]);
    k.sigN[i] = R(p.sigma[i][N - 1]);
    for (int j = 0; j < N; ++j) {
      const double s = p.sigma[i][j];
      k.beta2[i][j] = R(2.0 * 3.0 * s / p.eps);  // beta_ij = 3 sigma_ij / eps
      k.grad34[i][j] = R(0.75 * p.eps * s);
      k.wet3[i][j] = R(3.0 * s);
      k.inv_sig[i][j] = i == j ? R(0) : R(1.0 / s);
    }
  }
  double w[19];
  lattice_weights(p.lattice_f, p.d0, w);
  for (int q = 0; q < lattice_q(p.lattice_f); ++q) k.wf[q] = R(w[q]);
  lattice_weights(p.lattice_g, p.d0, w);
  for (int q = 0; q < lattice_q(p.lattice_g); ++q) k.wg[q] = R(w[q]);
  const double w0g = w[0];
  for (int r = 0; r < 6; ++r) {
    k.sf[r] = R(p.s_f[r]);
    k.sg[r] = R(p.s_g[r]);
  }
  k.two_over_c2mcs2 = R(2.0 / (1.0 - cs2));
  k.h2diag = R(1.0 / (cs2 - cs2 * cs2));
  k.h2off = R(1.0 / (cs2 * cs2));
  k.inv_c2mcs2 = R(1.0 / (1.0 - cs2));
  k.pref = R(cs2 / (1.0 - w0g));
  const double K = w0g / (1.0 - p.d0);  // eq. 19: 1 - d0 (2D), 1 - 2 d0 (3D)
  const double s0 = p.s_g[DDCC_S0];
  k.cgr = R(0.5 + K * (1.0 - p.d0) * (2.0 - s0) / (2.0 * s0));
  k.halfK = R(0.5 * K);
  k.KH = R(p.dim == 2 ? K * (1.0 - 2.0 * p.d0) : K * (3.0 - 7.0 * p.d0) / 2.0);
  k.one_m3cs2 = R(1.0 - 3.0 * cs2);
  for (int a = 0; a < 3; ++a) {
    k.accel[a] = R(p.accel[a]);
    k.force[a] = R(p.force[a]);
  }
  double q4[3][3];
  fourth_order_q(p.lattice_g, p.d0, q4);
  for (int j = 0; j < 3; ++j)
    for (int g = 0; g < 3; ++g) k.q4[j][g] = R(q4[j][g]);
}

template <class Pop, class S>
Bufs<Pop, S> bufs(ddcc_ctx* c, int mode) {
  Bufs<Pop, S> b{};
  const int a = c->cur, o = c->cur ^ 1;
  b.fA = static_cast<const Pop*>(c->f[a]);
  b.f0A = c->f0[a];
  b.gA = static_cast<const Pop*>(c->g[a]);
  b.TA = static_cast<const S*>(c->T[a]);
  if (mode == MODE_INIT) {
    b.fB = static_cast<Pop*>(c->f[a]);
    b.f0B = c->f0[a];
    b.gB = static_cast<Pop*>(c->g[a]);
    b.TB = static_cast<S*>(c->T[a]);
  } else {
    b.fB = static_cast<Pop*>(c->f[o]);
    b.f0B = c->f0[o];
    b.gB = static_cast<Pop*>(c->g[o]);
    b.TB = static_cast<S*>(c->T[o]);
  }
  b.hist = static_cast<S*>(c->hist);
  b.psi = static_cast<const S*>(c->psi);
  b.wet = static_cast<const S*>(c->wet);
  if (c->work) {
    b.fC = c->work;
    b.fmu = c->work + (size_t)c->p.nphase * c->n;
  }
  b.coef_d = c->dkd;
  b.coef_r = sizeof(S) == 8 ? static_cast<const void*>(c->dkd)
                            : static_cast<const void*>(c->dkf);
  return b;
}

template <class Pop, class S, class R>
hipError_t launch_as(ddcc_ctx* c, const Coef<R>& k, int mode,
                     const double* inC, const double* inU, const double* inP,
                     double* oC, double* oU, double* oP) {
  Bufs<Pop, S> b = bufs<Pop, S>(c, mode);
  if (mode == MODE_STEP && c->stream_stores)
    mode = c->p.dim == 2 && !rows_on_lines(c->p.nx, sizeof(Pop)) ? MODE_RAGGED
                                                                 : MODE_STREAM;
  b.inC = inC;
  b.inU = inU;
  b.inP = inP;
  b.outC = oC;
  b.outU = oU;
  b.outP = oP;
  if (c->p.dim == 2) {
    b.out_n = c->nodes;
    return launch_2d<Pop, S, R>(c->p.nphase, mode, c->kd, k, b, c->tile_y,
                                c->cus, c->stream);
  }
  return launch_3d<Pop, S, R>(c->p.nphase, c->p.lattice_f, mode, c->kd, k, b,
                              c->tile_x, c->tile_y, c->cus, c->stream);
}

hipError_t launch(ddcc_ctx* c, int mode, const double* inC, const double* inU,
                  const double* inP, double* oC, double* oU, double* oP) {
  switch (c->p.precision) {
    case DDCC_FP64:
      return launch_as<double, double>(c, c->kd, mode, inC, inU, inP, oC, oU,
                                       oP);
    case DDCC_FP16:
      return launch_as<_Float16, float>(c, c->kf, mode, inC, inU, inP, oC, oU,
                                        oP);
    case DDCC_BF16:
      return launch_as<__bf16, float>(c, c->kf, mode, inC, inU, inP, oC, oU,
                                      oP);
    default:
      return launch_as<float, float>(c, c->kf, mode, inC, inU, inP, oC, oU,
                                     oP);
  }
}

int ensure_staging(ddcc_ctx* c) {
  if (c->staging) return DDCC_OK;
  const size_t count = (size_t)(c->p.nphase + c->p.dim + 1) * c->nodes;
  HIPCHK(c, hipMalloc(&c->staging, count * sizeof(double)), "hipMalloc staging");
  return DDCC_OK;
}

bool all_finite(const double* a, size_t count) {
  for (size_t i = 0; i < count; ++i)
    if (!std::isfinite(a[i])) return false;
  return true;
}

// Steps of a small box in captured groups. A launch costs the host 2.5 to 4
// us, and a step of a box of up to kGraphNodes nodes 6 to 10 us of one stream
// (three launches in 3D): a program that runs a few such boxes at once waits
// for launches. A captured group costs about 18 us and 0.25 us per step. The
// groups are made once a context has run kGraphAfter steps one by one (making
// them costs as much as launching their steps, and the steps already queued
// cover it); every call starts with kGraphLead steps one by one, so that the
// device has work while the first group is handed over. Passes over three
// contexts in turn (same GPU): 96 x 70 FP32, 200 steps 774 -> 491 us; 128^2
// FP64, 100 steps 381 -> 321 us. One context alone waits for its kernels
// either way (96 x 70 FP32 6.6 -> 6.4 us per step).
constexpr long long kGraphNodes = 1 << 17;
constexpr int64_t kGraphAfter = 128;
constexpr int64_t kGraphLead = 8;
constexpr int kGraphSteps[2] = {64, 16};  // even: cur keeps its parity

void drop_step_graphs(ddcc_ctx* c) {
  for (auto& by_size : c->step_graph)
    for (auto& by_parity : by_size)
      for (hipGraphExec_t& g : by_parity)
        if (g) {
          (void)hipGraphExecDestroy(g);
          g = nullptr;
        }
}

// Whether steps may be launched as groups now: a small box, past its first
// steps, on a stream that the caller is not capturing.
bool graphs_usable(ddcc_ctx* c) {
  if (c->n > kGraphNodes || c->graphs_failed || c->direct_steps < kGraphAfter)
    return false;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) {
    (void)hipGetLastError();  // not the error of the launch that follows
    return false;
  }
  return st == hipStreamCaptureStatusNone;
}

// The captured group of kGraphSteps[q] steps from the current parity, made on
// a stream of the context's own (nothing else can be recorded there); nullptr
// if that failed. A group stays until the context is destroyed, so nothing
// here waits for the device, also after a change of the tile.
hipGraphExec_t step_graph(ddcc_ctx* c, int q) {
  const int by_tile =
      c->tile_y == 2 ? 0 : (c->tile_y == 4 ? 1 : (c->tile_y == 8 ? 2 : 3));
  hipGraphExec_t& exec = c->step_graph[by_tile][q][c->cur];
  if (exec || c->graphs_failed) return exec;
  // the calls below are allowed whatever else this thread captures
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  const ddcc::detail::OnDevice on(c->device);
  hipError_t e = on.status;
  if (e == hipSuccess && !c->capture_stream)
    e = hipStreamCreateWithFlags(&c->capture_stream, hipStreamNonBlocking);
  if (e == hipSuccess)
    e = hipStreamBeginCapture(c->capture_stream, hipStreamCaptureModeRelaxed);
  if (e == hipSuccess) {
    const hipStream_t stream = c->stream;
    const int cur = c->cur;
    c->stream = c->capture_stream;
    for (int s = 0; s < kGraphSteps[q] && e == hipSuccess; ++s) {
      e = launch(c, MODE_STEP, nullptr, nullptr, nullptr, nullptr, nullptr,
                 nullptr);
      c->cur ^= 1;
    }
    c->stream = stream;
    c->cur = cur;
    hipGraph_t graph = nullptr;
    const hipError_t end = hipStreamEndCapture(c->capture_stream, &graph);
    if (e == hipSuccess) e = end;
    if (e == hipSuccess)
      e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    if (graph) (void)hipGraphDestroy(graph);
  }
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    exec = nullptr;
    c->graphs_failed = true;
  }
  return exec;
}

// nsteps steps with nothing between them.
hipError_t run_steps(ddcc_ctx* c, int64_t nsteps) {
  const bool groups =
      nsteps >= kGraphLead + kGraphSteps[1] && graphs_usable(c);
  for (int64_t s = 0; s < nsteps;) {
    if (groups && s >= kGraphLead) {
      const int q = nsteps - s >= kGraphSteps[0] ? 0 : 1;
      const hipGraphExec_t g =
          nsteps - s >= kGraphSteps[q] ? step_graph(c, q) : nullptr;
      if (g) {
        if (hipGraphLaunch(g, c->stream) == hipSuccess) {
          s += kGraphSteps[q];
          c->t += kGraphSteps[q];
          continue;
        }
        // refused (a group's arguments take device memory): single launches,
        // which report what is wrong if they fail too
        (void)hipGetLastError();
        c->graphs_failed = true;
      }
    }
    const hipError_t e = launch(c, MODE_STEP, nullptr, nullptr, nullptr,
                                nullptr, nullptr, nullptr);
    if (e != hipSuccess) return e;
    c->cur ^= 1;
    ++c->t;
    ++c->direct_steps;
    ++s;
  }
  return hipSuccess;
}

void release(ddcc_ctx* c) {
  drop_step_graphs(c);
  if (c->capture_stream) (void)hipStreamDestroy(c->capture_stream);
  void* ptrs[] = {c->f[0],  c->f[1],   c->f0[0],    c->f0[1], c->g[0],
                  c->g[1],  c->T[0],   c->T[1],     c->hist,  c->psi,
                  c->wet,   c->staging, c->partial, c->bad,  c->work,
                  c->diag_partial, c->diag_first,
                  c->dkd,   c->dkf,    c->geo64};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  for (hipEvent_t e : c->adj_events)
    if (e) (void)hipEventDestroy(e);
  if (c->adj_stream) (void)hipStreamDestroy(c->adj_stream);
  if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
}

// Launch the per-phase population sums of the current state into
// partial[block * N + i] with non-finite flags bad[block]; *first = t at the
// first non-finite population if first is not NULL (launch_mass).
hipError_t mass_into(ddcc_ctx* c, double* partial, int* bad,
                     long long* first = nullptr, long long t = 0) {
  const int N = c->p.nphase;
  const void* f = c->f[c->cur];
  const double* f0 = c->f0[c->cur];
  const auto go = [&](const auto* pops) {
    return launch_mass(f0, pops, N, c->Qf, c->n, c->n, partial, bad,
                       c->mass_blocks, c->stream, first, t);
  };
  switch (c->p.precision) {
    case DDCC_FP64:
      return go(static_cast<const double*>(f));
    case DDCC_FP16:
      return go(static_cast<const _Float16*>(f));
    case DDCC_BF16:
      return go(static_cast<const __bf16*>(f));
    default:
      return go(static_cast<const float*>(f));
  }
}

// Clear the record of the periodic checks (new state or new setting).
int diag_reset(ddcc_ctx* c) {
  c->diag_t = -1;
  if (!c->diag_first) return DDCC_OK;
  const long long none = -1;
  HIPCHK(c, hipMemcpyAsync(c->diag_first, &none, sizeof(none),
                           hipMemcpyHostToDevice, c->stream),
         "clear diagnostics");
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  return DDCC_OK;
}

// The arrays of a checkpoint in its order; on the host their rows are nx nodes
// long, on the device px.
struct StatePart {
  void* dev;
  size_t planes, esz;
};

std::array<StatePart, 5> state_parts(ddcc_ctx* c) {
  const size_t N = (size_t)c->p.nphase;
  return {StatePart{c->f[c->cur], N * (size_t)(c->Qf - 1), c->pesz},
          StatePart{c->f0[c->cur], N, sizeof(double)},
          StatePart{c->g[c->cur], (size_t)c->Qg, c->pesz},
          StatePart{c->hist, (size_t)c->nhist, c->esz},
          StatePart{c->T[c->cur], (size_t)c->nT, c->esz}};
}

// Copy a part to the host (to) or from it. Padded rows go through the work
// fields, which hold nothing between steps, as many planes at a time as fit
// (the copy engine's own pitched copy of 248 MB took 3.1 s, this one 24 ms).
hipError_t copy_part(ddcc_ctx* c, const StatePart& q, char* to,
                     const char* from) {
  const hipMemcpyKind kind = to ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice;
  if (c->px == c->p.nx) {
    const size_t bytes = q.planes * (size_t)c->n * q.esz;
    if (to) return hipMemcpyAsync(to, q.dev, bytes, kind, c->stream);
    return hipMemcpyAsync(q.dev, from, bytes, kind, c->stream);
  }
  const size_t fit = 2 * (size_t)c->p.nphase * sizeof(double) / q.esz;
  for (size_t i = 0; i < q.planes; i += fit) {
    const size_t m = q.planes - i < fit ? q.planes - i : fit;
    const long long rows = (long long)m * c->p.ny * c->p.nz;
    const size_t bytes = m * (size_t)c->nodes * q.esz;
    const size_t at = i * (size_t)c->nodes * q.esz;
    char* dev = static_cast<char*>(q.dev) + i * (size_t)c->n * q.esz;
    hipError_t e = hipSuccess;
    if (!to) e = hipMemcpyAsync(c->work, from + at, bytes, kind, c->stream);
    if (e == hipSuccess)
      e = launch_copy_rows(dev, c->work, to != nullptr, c->p.nx, c->px, rows,
                           q.esz, c->stream);
    if (e == hipSuccess && to)
      e = hipMemcpyAsync(to + at, c->work, bytes, kind, c->stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

struct SaveHeader {
  char magic[8];
  int32_t dim, nx, ny, nz, nphase, lattice_f, lattice_g, precision;
  int64_t t;
  int64_t bytes;
};

}  // namespace

namespace ddcc {
bool have_3d();

namespace detail {
int fail(ddcc_ctx* c, int code, const std::string& msg) {
  return ::fail(c, code, msg);
}
int hip_fail(ddcc_ctx* c, hipError_t e, const char* what) {
  return ::hip_fail(c, e, what);
}
hipError_t step_launch(ddcc_ctx* c) {
  return launch(c, MODE_STEP, nullptr, nullptr, nullptr, nullptr, nullptr,
                nullptr);
}
}  // namespace detail
}  // namespace ddcc

extern "C" {

const char* ddcc_version(void) { return kVersion; }

int ddcc_default_params(ddcc_params* p) {
  if (!p) return DDCC_E_INVAL;
  std::memset(p, 0, sizeof(*p));
  p->dim = 2;
  p->nx = 64;
  p->ny = 64;
  p->nz = 1;
  p->nphase = 2;
  p->lattice_f = DDCC_D2Q9;
  p->lattice_g = DDCC_D2Q9;
  p->precision = DDCC_FP64;
  p->d0 = 0.4;
  p->eps = 5.0;
  p->m0 = 0.05;
  p->rho0 = 1.0;
  p->psi_min = 1e-30;
  p->lam = 1.0 / std::pow(2.0 * std::sqrt(2.0) * 1.5, 3);
  for (int i = 0; i < DDCC_MAX_PHASES; ++i) {
    p->rho[i] = 1.0;
    p->nu[i] = 0.1;
    p->eta[i] = 0.0;
    for (int j = 0; j < DDCC_MAX_PHASES; ++j)
      p->sigma[i][j] = i == j ? 0.0 : 0.001;
  }
  const double sf[6] = {1.0, 10.0 / 19.0, 1.2, 1.2, 1.2, 1.2};
  const double sg[6] = {1.0, 1.2, 1.2, 1.2, 1.2, 1.2};
  for (int r = 0; r < 6; ++r) {
    p->s_f[r] = sf[r];
    p->s_g[r] = sg[r];
  }
  return DDCC_OK;
}

// A context of validated parameters whose rows are px nodes apart.
static int create_with_pitch(const ddcc_params* p, int px, void* stream,
                             ddcc_ctx** out) {
  ddcc_ctx* c = new (std::nothrow) ddcc_ctx();
  if (!c) return DDCC_E_NOMEM;
  c->p = *p;
  c->nodes = (long long)p->nx * p->ny * p->nz;
  c->px = px;
  c->n = (long long)c->px * p->ny * p->nz;
  c->Qf = lattice_q(p->lattice_f);
  c->Qg = lattice_q(p->lattice_g);
  const int d = p->dim;
  // 2D: phi C_i u (2N), Y (3), P; 3D: phi C_i (N), u (3), m^C (3), P
  c->nhist = d == 2 ? 2 * p->nphase + 4 : p->nphase + 7;
  c->nT = d * (d - 1) / 2;
  c->esz = field_bytes(*p);
  c->pesz = pop_bytes(*p);
  if (hipGetDevice(&c->device) != hipSuccess ||
      hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount,
                            c->device) != hipSuccess) {
    delete c;
    return DDCC_E_HIP;
  }
  // 3D: 64 x 4 columns
  c->tile_y =
      d == 2 ? default_tile_2d(p->nx, p->ny, p->nphase, c->pesz, c->cus) : 4;
  c->tile_x = 64;
  if (stream) {
    c->stream = static_cast<hipStream_t>(stream);
  } else {
    if (hipStreamCreate(&c->stream) != hipSuccess) {
      delete c;
      return DDCC_E_HIP;
    }
    c->own_stream = true;
  }
  fill_coef<double>(c->p, c->px, c->n, c->kd);
  fill_coef<float>(c->p, c->px, c->n, c->kf);
  const size_t n = (size_t)c->n;
  const size_t sf = (size_t)p->nphase * (c->Qf - 1) * n * c->pesz;
  const size_t sg = (size_t)c->Qg * n * c->pesz;
  const size_t sT = (size_t)c->nT * n * c->esz;
  hipError_t e = hipSuccess;
  for (int a = 0; a < 2 && e == hipSuccess; ++a) {
    e = hipMalloc(&c->f[a], sf);
    if (e == hipSuccess)
      e = hipMalloc(&c->f0[a], (size_t)p->nphase * n * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&c->g[a], sg);
    if (e == hipSuccess) e = hipMalloc(&c->T[a], sT);
  }
  if (e == hipSuccess) e = hipMalloc(&c->hist, (size_t)c->nhist * n * c->esz);
  c->stream_stores = step_bytes_of(*p, n) > kCacheBytes;
  if (e == hipSuccess) e = hipMalloc(&c->psi, n * c->esz);
  if (e == hipSuccess)
    e = hipMalloc(&c->wet, (size_t)(p->nphase - 1) * n * c->esz);
  if (e == hipSuccess && p->dim == 3)
    e = hipMalloc(&c->work, (size_t)2 * p->nphase * n * sizeof(double));
  long long mb = (c->n + 255) / 256;
  c->mass_blocks = (int)(mb > kScratchBlocks ? kScratchBlocks : mb);
  if (e == hipSuccess)
    e = hipMalloc(&c->partial,
                  (size_t)c->mass_blocks * p->nphase * sizeof(double));
  if (e == hipSuccess) e = hipMalloc(&c->bad, (size_t)c->mass_blocks * sizeof(int));
  if (e == hipSuccess) e = hipMalloc(&c->dkd, sizeof(Coef<double>));
  if (e == hipSuccess) e = hipMalloc(&c->dkf, sizeof(Coef<float>));
  if (e == hipSuccess)
    e = hipMemcpy(c->dkd, &c->kd, sizeof(Coef<double>), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(c->dkf, &c->kf, sizeof(Coef<float>), hipMemcpyHostToDevice);
  // no kernel touches the padding of the rows but the mass sums, which take
  // it with the nodes
  for (int a = 0; a < 2 && e == hipSuccess && c->px != p->nx; ++a) {
    e = hipMemsetAsync(c->f[a], 0, sf, c->stream);
    if (e == hipSuccess)
      e = hipMemsetAsync(c->f0[a], 0, (size_t)p->nphase * n * sizeof(double),
                         c->stream);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();  // see hip_fail
    release(c);
    delete c;
    return e == hipErrorOutOfMemory ? DDCC_E_NOMEM : DDCC_E_HIP;
  }
  if (p->dim == 3) {
    // The 3D kernels are built per (phase, flow) lattice pair; the host
    // checks the pair here so that create fails early when it is absent.
    if (!((p->lattice_f == DDCC_D3Q15 || p->lattice_f == DDCC_D3Q7) &&
          p->lattice_g == DDCC_D3Q19) ||
        p->nphase > 3 || !have_3d()) {
      release(c);
      delete c;
      return DDCC_E_UNSUPPORTED;
    }
  }
  *out = c;
  return DDCC_OK;
}

int ddcc_create(const ddcc_params* p, void* stream, ddcc_ctx** out) {
  if (!out) return DDCC_E_INVAL;
  *out = nullptr;
  std::string msg;
  int rc = validate(p, msg);
  if (rc != DDCC_OK) return rc;
  const int px = row_pitch(*p);
  rc = create_with_pitch(p, px, stream, out);
  // padded rows are for speed alone: where they do not fit, dense ones may
  if (rc == DDCC_E_NOMEM && px != p->nx)
    rc = create_with_pitch(p, p->nx, stream, out);
  return rc;
}

static int ensure_geo64(ddcc_ctx* c) {
  if (c->geo64) return DDCC_OK;
  const size_t count = (size_t)c->p.nphase * c->n;
  HIPCHK(c, hipMalloc(&c->geo64, count * sizeof(double)),
         "hipMalloc float64 geometry");
  return DDCC_OK;
}

// Geometry of K walls from float64 device arrays psik [K][n] and ctk
// [K][N-1][n] (NULL: 90 degrees): psi and the wetting weights in the
// context's field precision.
static int geometry_from_device(ddcc_ctx* c, int K, const double* psik,
                                const double* ctk) {
  const int nm1 = c->p.nphase - 1;
  hipError_t e =
      c->p.precision == DDCC_FP64
          ? launch_wet_field<double>(psik, ctk, K, nm1, c->p.nx, c->p.ny,
                                     c->p.nz, c->px, static_cast<double*>(c->psi),
                                     static_cast<double*>(c->wet), c->n, 0,
                                     c->stream)
          : launch_wet_field<float>(psik, ctk, K, nm1, c->p.nx, c->p.ny,
                                    c->p.nz, c->px, static_cast<float*>(c->psi),
                                    static_cast<float*>(c->wet), c->n, 0,
                                    c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "geometry kernel");
  // The adjoint's derivative of the wetting weights E_i = cos theta_iN
  // |grad psi| with respect to psi is cos theta_iN grad psi / |grad psi|,
  // taken from the float64 psi and cosines: a float32 psi rounds to 1 a few
  // cells off a wall, where grad psi is small but not zero, and E_i / |grad
  // psi| mixes two evaluations of |grad psi| that differ in their rounding
  // where psi is 1 up to rounding. 2D contexts with one wall (those the
  // adjoint supports) keep the float64 psi and cosines.
  if (c->p.dim == 2 && K == 1) {
    const size_t n = (size_t)c->n;
    const int rc = ensure_geo64(c);
    if (rc) return rc;
    e = hipMemcpyAsync(c->geo64, psik, n * sizeof(double),
                       hipMemcpyDeviceToDevice, c->stream);
    if (e == hipSuccess)
      e = ctk ? hipMemcpyAsync(c->geo64 + n, ctk, nm1 * n * sizeof(double),
                               hipMemcpyDeviceToDevice, c->stream)
              : hipMemsetAsync(c->geo64 + n, 0, nm1 * n * sizeof(double),
                               c->stream);
    if (e != hipSuccess) return hip_fail(c, e, "copy float64 geometry");
  }
  c->geom_ok = true;
  c->nwalls = K;
  c->fields_ok = false;
  return DDCC_OK;
}

// Checks K walls on the host (psi_k in [0, 1], cosines in [-1, 1]).
static int check_walls(ddcc_ctx* c, int K, const double* psik,
                       const double* ctk) {
  if (K < 1 || K > DDCC_MAX_WALLS)
    return fail(c, DDCC_E_INVAL, "number of walls must be in [1, 8]");
  if (!psik) return fail(c, DDCC_E_INVAL, "psi is NULL");
  const size_t n = (size_t)c->nodes;
  for (size_t i = 0; i < (size_t)K * n; ++i)
    if (!(psik[i] >= 0.0 && psik[i] <= 1.0))
      return fail(c, DDCC_E_INVAL, "psi must be finite and in [0, 1]");
  if (ctk)
    for (size_t i = 0; i < (size_t)K * (c->p.nphase - 1) * n; ++i)
      if (!(ctk[i] >= -1.0 && ctk[i] <= 1.0))
        return fail(c, DDCC_E_INVAL, "cos_theta must be finite and in [-1, 1]");
  return DDCC_OK;
}

int ddcc_init_geometry_walls(ddcc_ctx* c, int nwalls, const double* psi,
                             const double* cos_theta) {
  if (!c) return DDCC_E_INVAL;
  int rc = check_walls(c, nwalls, psi, cos_theta);
  if (rc) return rc;
  const size_t n = (size_t)c->nodes, np = (size_t)nwalls * n;
  const size_t nc = cos_theta ? np * (c->p.nphase - 1) : 0;
  // Boxes of up to kKeepNodes nodes keep the staging memory that init_fields
  // uses too; larger ones, and walls that do not fit it, take their own for
  // the call. (hipFree waits for every stream of the device: where geometry is
  // set in a loop, as a fit of the angles does, the call took 2.9 ms instead
  // of 0.1 after other streams' work, 256^2.)
  constexpr long long kKeepNodes = 1 << 20;
  const size_t room = (size_t)(c->p.nphase + c->p.dim + 1) * n;
  bool keep = c->nodes <= kKeepNodes && np + nc <= room;
  double* d = nullptr;
  if (keep) {
    // what the geometry needs anyway comes first
    if (c->p.dim == 2 && nwalls == 1 && (rc = ensure_geo64(c))) return rc;
    rc = ensure_staging(c);
    if (rc && rc != DDCC_E_NOMEM) return rc;
    keep = rc == DDCC_OK;  // else there may be room for the walls alone
    d = c->staging;
  }
  if (!keep) {
    HIPCHK(c, hipMalloc(&d, (np + nc) * sizeof(double)), "hipMalloc geometry");
  }
  hipError_t e = hipMemcpyAsync(d, psi, np * sizeof(double),
                                hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess && nc)
    e = hipMemcpyAsync(d + np, cos_theta, nc * sizeof(double),
                       hipMemcpyHostToDevice, c->stream);
  if (e != hipSuccess) {
    if (!keep) (void)hipFree(d);
    return hip_fail(c, e, "copy geometry");
  }
  rc = geometry_from_device(c, nwalls, d, nc ? d + np : nullptr);
  e = hipStreamSynchronize(c->stream);
  if (!keep) (void)hipFree(d);
  if (rc) return rc;
  if (e != hipSuccess) return hip_fail(c, e, "sync");
  return DDCC_OK;
}

int ddcc_init_geometry(ddcc_ctx* c, const double* psi, const double* ct) {
  return ddcc_init_geometry_walls(c, 1, psi, ct);
}

int ddcc_init_geometry_dev(ddcc_ctx* c, const double* psi, const double* ct) {
  if (!c) return DDCC_E_INVAL;
  if (!psi) return fail(c, DDCC_E_INVAL, "psi is NULL");
  return geometry_from_device(c, 1, psi, ct);
}

static int init_fields_common(ddcc_ctx* c, const double* C, const double* u,
                              const double* P) {
  hipError_t e = launch(c, MODE_INIT, C, u, P, nullptr, nullptr, nullptr);
  if (e != hipSuccess) return hip_fail(c, e, "init kernel");
  c->fields_ok = true;
  c->t = 0;
  return diag_reset(c);
}

int ddcc_init_fields(ddcc_ctx* c, const double* C, const double* u,
                     const double* P) {
  if (!c) return DDCC_E_INVAL;
  if (!c->geom_ok) return fail(c, DDCC_E_STATE, "init_geometry first");
  if (!C) return fail(c, DDCC_E_INVAL, "C is NULL");
  const size_t n = (size_t)c->nodes;
  const int N = c->p.nphase, d = c->p.dim;
  if (!all_finite(C, N * n) || (u && !all_finite(u, d * n)) ||
      (P && !all_finite(P, n)))
    return fail(c, DDCC_E_INVAL, "non-finite initial field");
  int rc = ensure_staging(c);
  if (rc) return rc;
  double* sC = c->staging;
  double* sU = sC + N * n;
  double* sP = sU + d * n;
  HIPCHK(c, hipMemcpyAsync(sC, C, N * n * sizeof(double), hipMemcpyHostToDevice,
                           c->stream),
         "copy C");
  if (u)
    HIPCHK(c, hipMemcpyAsync(sU, u, d * n * sizeof(double),
                             hipMemcpyHostToDevice, c->stream),
           "copy u");
  if (P)
    HIPCHK(c, hipMemcpyAsync(sP, P, n * sizeof(double), hipMemcpyHostToDevice,
                             c->stream),
           "copy P");
  rc = init_fields_common(c, sC, u ? sU : nullptr, P ? sP : nullptr);
  if (rc) return rc;
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  return DDCC_OK;
}

int ddcc_init_fields_dev(ddcc_ctx* c, const double* C, const double* u,
                         const double* P) {
  if (!c) return DDCC_E_INVAL;
  if (!c->geom_ok) return fail(c, DDCC_E_STATE, "init_geometry first");
  if (!C) return fail(c, DDCC_E_INVAL, "C is NULL");
  return init_fields_common(c, C, u, P);
}

int ddcc_step(ddcc_ctx* c, int64_t nsteps) {
  if (!c) return DDCC_E_INVAL;
  if (nsteps < 0) return fail(c, DDCC_E_INVAL, "nsteps < 0");
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  for (int64_t left = nsteps; left > 0;) {
    int64_t k = left;  // up to the next check
    if (c->diag_every > 0) {
      const int64_t gap = c->diag_every - c->t % c->diag_every;
      if (gap < k) k = gap;
    }
    hipError_t e = run_steps(c, k);
    if (e != hipSuccess) return hip_fail(c, e, "step kernel");
    left -= k;
    if (c->diag_every > 0 && c->t % c->diag_every == 0) {
      e = mass_into(c, c->diag_partial, nullptr, c->diag_first,
                    (long long)c->t);
      if (e != hipSuccess) return hip_fail(c, e, "diagnostics");
      c->diag_t = c->t;
    }
  }
  return DDCC_OK;
}

static int moments_common(ddcc_ctx* c, double* C, double* u, double* P) {
  hipError_t e = launch(c, MODE_MOMENTS, nullptr, nullptr, nullptr, C, u, P);
  if (e != hipSuccess) return hip_fail(c, e, "moments kernel");
  return DDCC_OK;
}

int ddcc_read_moments(ddcc_ctx* c, double* C, double* u, double* P) {
  if (!c) return DDCC_E_INVAL;
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  int rc = ensure_staging(c);
  if (rc) return rc;
  const size_t n = (size_t)c->nodes;
  const int N = c->p.nphase, d = c->p.dim;
  double* sC = c->staging;
  double* sU = sC + N * n;
  double* sP = sU + d * n;
  rc = moments_common(c, sC, sU, sP);
  if (rc) return rc;
  if (C)
    HIPCHK(c, hipMemcpyAsync(C, sC, N * n * sizeof(double),
                             hipMemcpyDeviceToHost, c->stream),
           "copy C");
  if (u)
    HIPCHK(c, hipMemcpyAsync(u, sU, d * n * sizeof(double),
                             hipMemcpyDeviceToHost, c->stream),
           "copy u");
  if (P)
    HIPCHK(c, hipMemcpyAsync(P, sP, n * sizeof(double), hipMemcpyDeviceToHost,
                             c->stream),
           "copy P");
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  return DDCC_OK;
}

int ddcc_read_moments_dev(ddcc_ctx* c, double* C, double* u, double* P) {
  if (!c) return DDCC_E_INVAL;
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  if (!C || !u || !P)
    return fail(c, DDCC_E_INVAL, "device read-out needs all three outputs");
  return moments_common(c, C, u, P);
}

int ddcc_mass(ddcc_ctx* c, double* mass) {
  if (!c || !mass) return fail(c, DDCC_E_INVAL, "NULL argument");
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  const int N = c->p.nphase;
  const hipError_t e = mass_into(c, c->partial, c->bad);
  if (e != hipSuccess) return hip_fail(c, e, "mass kernel");
  std::vector<double> part((size_t)c->mass_blocks * N);
  std::vector<int> bad(c->mass_blocks);
  HIPCHK(c, hipMemcpyAsync(part.data(), c->partial, part.size() * sizeof(double),
                           hipMemcpyDeviceToHost, c->stream),
         "copy partials");
  HIPCHK(c, hipMemcpyAsync(bad.data(), c->bad, bad.size() * sizeof(int),
                           hipMemcpyDeviceToHost, c->stream),
         "copy flags");
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  for (int i = 0; i < N; ++i) {
    double s = 0.0;
    for (int b = 0; b < c->mass_blocks; ++b) s += part[(size_t)b * N + i];
    mass[i] = s;
  }
  for (int b = 0; b < c->mass_blocks; ++b)
    if (bad[b]) return fail(c, DDCC_E_NONFINITE, "non-finite population");
  return DDCC_OK;
}

int ddcc_mass_noalloc(ddcc_ctx* c, double* mass_dev, int* nonfinite_dev) {
  if (!c || !mass_dev) return fail(c, DDCC_E_INVAL, "NULL argument");
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  const int N = c->p.nphase;
  void* ws = nullptr;
  size_t cap = 0;
  HIPCHK(c, scratch_address(c->device, &ws, &cap), "static workspace address");
  const size_t part_bytes = (size_t)kScratchBlocks * kMaxN * sizeof(double);
  const size_t need_part = (size_t)c->mass_blocks * N * sizeof(double);
  const size_t need_bad = (size_t)c->mass_blocks * sizeof(int);
  if (c->mass_blocks > kScratchBlocks || need_part > part_bytes ||
      part_bytes + need_bad > cap)
    return fail(c, DDCC_E_INVAL,
                "mass check needs more than the static workspace (1024 "
                "blocks of partial sums)");
  double* partial = static_cast<double*>(ws);
  int* bad = reinterpret_cast<int*>(static_cast<char*>(ws) + part_bytes);
  hipError_t e = mass_into(c, partial, bad);
  if (e == hipSuccess)
    e = launch_mass_finish(partial, bad, c->mass_blocks, N, mass_dev,
                           nonfinite_dev, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "mass kernel");
  return DDCC_OK;
}

int64_t ddcc_time(const ddcc_ctx* c) { return c ? c->t : -1; }

int ddcc_save(ddcc_ctx* c, void* buf, size_t* bytes) {
  if (!c || !bytes) return fail(c, DDCC_E_INVAL, "NULL argument");
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  const size_t n = (size_t)c->nodes;
  const size_t sf = (size_t)c->p.nphase * (c->Qf - 1) * n * c->pesz;
  const size_t sg = (size_t)c->Qg * n * c->pesz;
  const size_t sh = (size_t)c->nhist * n * c->esz;
  const size_t sT = (size_t)c->nT * n * c->esz;
  const size_t s0 = (size_t)c->p.nphase * n * sizeof(double);
  const size_t need = sizeof(SaveHeader) + sf + s0 + sg + sh + sT;
  if (!buf) {
    *bytes = need;
    return DDCC_OK;
  }
  if (*bytes < need) return fail(c, DDCC_E_INVAL, "buffer too small");
  SaveHeader h{};
  std::memcpy(h.magic, "DDCCSAV4", 8);
  h.dim = c->p.dim;
  h.nx = c->p.nx;
  h.ny = c->p.ny;
  h.nz = c->p.nz;
  h.nphase = c->p.nphase;
  h.lattice_f = c->p.lattice_f;
  h.lattice_g = c->p.lattice_g;
  h.precision = c->p.precision;
  h.t = c->t;
  h.bytes = (int64_t)need;
  char* o = static_cast<char*>(buf);
  std::memcpy(o, &h, sizeof(h));
  o += sizeof(h);
  for (const StatePart& q : state_parts(c)) {
    HIPCHK(c, copy_part(c, q, o, nullptr), "save state");
    o += q.planes * n * q.esz;
  }
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  *bytes = need;
  return DDCC_OK;
}

int ddcc_load(ddcc_ctx* c, const void* buf, size_t bytes) {
  if (!c || !buf) return fail(c, DDCC_E_INVAL, "NULL argument");
  if (!c->geom_ok) return fail(c, DDCC_E_STATE, "init_geometry first");
  const size_t n = (size_t)c->nodes;
  const size_t sf = (size_t)c->p.nphase * (c->Qf - 1) * n * c->pesz;
  const size_t sg = (size_t)c->Qg * n * c->pesz;
  const size_t sh = (size_t)c->nhist * n * c->esz;
  const size_t sT = (size_t)c->nT * n * c->esz;
  const size_t s0 = (size_t)c->p.nphase * n * sizeof(double);
  const size_t need = sizeof(SaveHeader) + sf + s0 + sg + sh + sT;
  if (bytes < need) return fail(c, DDCC_E_INVAL, "checkpoint too small");
  SaveHeader h;
  std::memcpy(&h, buf, sizeof(h));
  if (std::memcmp(h.magic, "DDCCSAV4", 8) != 0 || h.dim != c->p.dim ||
      h.nx != c->p.nx || h.ny != c->p.ny || h.nz != c->p.nz ||
      h.nphase != c->p.nphase || h.lattice_f != c->p.lattice_f ||
      h.lattice_g != c->p.lattice_g || h.precision != c->p.precision ||
      h.bytes != (int64_t)need)
    return fail(c, DDCC_E_INVAL, "checkpoint does not match this context");
  const char* s = static_cast<const char*>(buf) + sizeof(h);
  for (const StatePart& q : state_parts(c)) {
    HIPCHK(c, copy_part(c, q, nullptr, s), "load state");
    s += q.planes * n * q.esz;
  }
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  c->t = h.t;
  c->fields_ok = true;
  return diag_reset(c);
}

int ddcc_sync(ddcc_ctx* c) {
  if (!c) return DDCC_E_INVAL;
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  if (c->diag_every > 0) {
    long long first = -1;
    HIPCHK(c, hipMemcpy(&first, c->diag_first, sizeof(first),
                        hipMemcpyDeviceToHost),
           "read diagnostics");
    if (first >= 0)
      return fail(c, DDCC_E_NONFINITE,
                  "non-finite population found by the check at step " +
                      std::to_string(first));
  }
  return DDCC_OK;
}

int ddcc_set_diagnostics(ddcc_ctx* c, int every) {
  if (!c) return DDCC_E_INVAL;
  if (every < 0) return fail(c, DDCC_E_INVAL, "every < 0");
  if (every > 0 && !c->diag_first) {
    const int N = c->p.nphase;
    HIPCHK(c, hipMalloc(&c->diag_partial,
                        (size_t)c->mass_blocks * N * sizeof(double)),
           "hipMalloc diagnostics");
    HIPCHK(c, hipMalloc(&c->diag_first, sizeof(long long)), "hipMalloc diagnostics");
  }
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  c->diag_every = every;
  return diag_reset(c);
}

int ddcc_diagnostics(ddcc_ctx* c, double* mass, int64_t* t_checked,
                     int64_t* t_nonfinite) {
  if (!c) return DDCC_E_INVAL;
  if (c->diag_every <= 0)
    return fail(c, DDCC_E_STATE, "diagnostics are off (ddcc_set_diagnostics)");
  const int N = c->p.nphase;
  std::vector<double> part((size_t)c->mass_blocks * N);
  long long first = -1;
  HIPCHK(c, hipStreamSynchronize(c->stream), "sync");
  if (c->diag_t >= 0 && mass)
    HIPCHK(c, hipMemcpy(part.data(), c->diag_partial,
                        part.size() * sizeof(double), hipMemcpyDeviceToHost),
           "read diagnostics");
  HIPCHK(c, hipMemcpy(&first, c->diag_first, sizeof(first),
                      hipMemcpyDeviceToHost),
         "read diagnostics");
  if (mass)
    for (int i = 0; i < N; ++i) {
      double sum = 0.0;
      for (int b = 0; b < c->mass_blocks; ++b) sum += part[(size_t)b * N + i];
      mass[i] = c->diag_t >= 0 ? sum : std::nan("");
    }
  if (t_checked) *t_checked = c->diag_t;
  if (t_nonfinite) *t_nonfinite = first;
  return DDCC_OK;
}

int ddcc_set_tile(ddcc_ctx* c, int tx, int ty) {
  if (!c) return DDCC_E_INVAL;
  if (c->p.dim == 2) {
    if (tx != 0 && tx != 64)
      return fail(c, DDCC_E_INVAL, "2D tiles are 64 nodes wide");
    if (ty != 0 && ty != 2 && ty != 4 && ty != 8 && ty != 16)
      return fail(c, DDCC_E_INVAL, "2D tile height must be 2, 4, 8 or 16");
    if (ty) c->tile_y = ty;
  } else {
    if (tx != 0 && tx != 64)
      return fail(c, DDCC_E_INVAL, "3D tiles are 64 nodes wide");
    if (ty != 0 && ty != 2 && ty != 4)
      return fail(c, DDCC_E_INVAL, "3D tile height must be 2 or 4");
    if (tx) c->tile_x = tx;
    if (ty) c->tile_y = ty;
  }
  return DDCC_OK;
}

int ddcc_autotune(ddcc_ctx* c, int steps, int* ty_out) {
  if (!c) return DDCC_E_INVAL;
  if (steps < 1) return fail(c, DDCC_E_INVAL, "steps < 1");
  if (!c->fields_ok) return fail(c, DDCC_E_STATE, "init_fields first");
  // The trial steps change the state: keep a copy of the current level (a
  // step reads populations and T at cur, writes them at cur ^ 1, and updates
  // the history in place).
  const size_t n = (size_t)c->n;
  const int N = c->p.nphase;
  const int cur0 = c->cur;
  const size_t sizes[5] = {(size_t)N * (c->Qf - 1) * n * c->pesz,
                           (size_t)N * n * sizeof(double),
                           (size_t)c->Qg * n * c->pesz,
                           (size_t)c->nT * n * c->esz,
                           (size_t)c->nhist * n * c->esz};
  void* src[5] = {c->f[cur0], c->f0[cur0], c->g[cur0], c->T[cur0], c->hist};
  void* keep[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  hipError_t e = hipSuccess;
  for (int q = 0; q < 5 && e == hipSuccess; ++q) {
    if (!sizes[q] || !src[q]) continue;
    e = hipMalloc(&keep[q], sizes[q]);
    if (e == hipSuccess)
      e = hipMemcpyAsync(keep[q], src[q], sizes[q], hipMemcpyDeviceToDevice,
                         c->stream);
  }
  const int cands2[4] = {2, 4, 8, 16}, cands3[2] = {2, 4};
  const int* cands = c->p.dim == 2 ? cands2 : cands3;
  const int ncand = c->p.dim == 2 ? 4 : 2;
  const int ty0 = c->tile_y;
  float best_ms = 0;
  int best = ty0;
  hipEvent_t t0 = nullptr, t1 = nullptr;
  if (e == hipSuccess) e = hipEventCreate(&t0);
  if (e == hipSuccess) e = hipEventCreate(&t1);
  const int64_t tsave = c->t;
  for (int k = 0; k < ncand && e == hipSuccess; ++k) {
    c->tile_y = cands[k];
    for (int s = 0; s < 2 + steps && e == hipSuccess; ++s) {
      if (s == 2) e = hipEventRecord(t0, c->stream);
      if (e == hipSuccess)
        e = launch(c, MODE_STEP, nullptr, nullptr, nullptr, nullptr, nullptr,
                   nullptr);
      c->cur ^= 1;
    }
    if (e == hipSuccess) e = hipEventRecord(t1, c->stream);
    if (e == hipSuccess) e = hipEventSynchronize(t1);
    float ms = 0;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, t0, t1);
    if (e == hipSuccess && (k == 0 || ms < best_ms)) {
      best_ms = ms;
      best = cands[k];
    }
  }
  // restore the level the trials started from
  c->cur = cur0;
  c->t = tsave;
  for (int q = 0; q < 5; ++q)
    if (keep[q] && e == hipSuccess)
      e = hipMemcpyAsync(src[q], keep[q], sizes[q], hipMemcpyDeviceToDevice,
                         c->stream);
  const hipError_t es = hipStreamSynchronize(c->stream);
  if (e == hipSuccess) e = es;
  for (int q = 0; q < 5; ++q)
    if (keep[q]) (void)hipFree(keep[q]);
  if (t0) (void)hipEventDestroy(t0);
  if (t1) (void)hipEventDestroy(t1);
  if (e != hipSuccess) {
    c->tile_y = ty0;
    return hip_fail(c, e, "autotune");
  }
  c->tile_y = best;
  if (ty_out) *ty_out = best;
  return DDCC_OK;
}

const char* ddcc_last_error(const ddcc_ctx* c) {
  return c ? c->err.c_str() : "NULL context";
}

void ddcc_destroy(ddcc_ctx* c) {
  if (!c) return;
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  release(c);
  delete c;
}

}  // extern "C"

// ===========================================================================
// Batches: many independent 2D D2Q9 boxes advanced by one launch per step.
// ===========================================================================
struct ddcc_batch {
  ddcc_params p{};
  int count = 0;
  std::vector<int> nx, ny;
  std::vector<long long> n, off;  // nodes and first node of each instance
  long long ntot = 0;             // plane stride: nodes of all instances
  hipStream_t stream = nullptr;
  bool own_stream = false;
  size_t esz = 8, pesz = 8;
  void* f[2] = {nullptr, nullptr};
  double* f0[2] = {nullptr, nullptr};
  void* g[2] = {nullptr, nullptr};
  void* T[2] = {nullptr, nullptr};
  void* hist = nullptr;
  void* psi = nullptr;
  void* wet = nullptr;        // wetting weights [N-1][ntot]
  double* staging = nullptr;  // (N + 3) planes of ntot float64
  double* partial = nullptr;
  int* bad = nullptr;
  int mass_blocks = 0;
  BatchTile* tiles = nullptr;
  BatchInst* insts = nullptr;
  std::vector<unsigned> t0, t1;  // tile range of each instance
  unsigned ntiles = 0;
  int ty = 8;
  int graph_steps = 0;           // 0: one launch per step, no graph
  bool stream_stores = false;    // steps as MODE_STREAM (see ddcc_ctx)
  hipGraphExec_t gexec[2] = {nullptr, nullptr};  // by parity of cur
  int cur = 0;
  std::vector<char> geom_ok, fields_ok;
  int64_t t = 0;
  std::string err;
  Coef<double> kd{};
  Coef<float> kf{};
  // device tables of every instance's coefficients (the batch parameters,
  // or an instance's own ones from ddcc_batch_set_params)
  Coef<double>* kds = nullptr;
  Coef<float>* kfs = nullptr;
};

namespace {

constexpr int kMaxGraphSteps = 1024;
constexpr int kBatchQ = 9;

int bfail(ddcc_batch* b, int code, const std::string& msg) {
  if (b) b->err = msg;
  return code;
}

int bhip(ddcc_batch* b, hipError_t e, const char* what) {
  (void)hipGetLastError();  // see hip_fail
  return bfail(b, e == hipErrorOutOfMemory ? DDCC_E_NOMEM : DDCC_E_HIP,
               std::string(what) + ": " + hipGetErrorString(e));
}

#define BHIP(b, expr, what)                            \
  do {                                                 \
    hipError_t e_ = (expr);                            \
    if (e_ != hipSuccess) return bhip(b, e_, what);    \
  } while (0)

int nhist_of(int N) { return 2 * N + 4; }

void drop_graphs(ddcc_batch* b) {
  for (auto& g : b->gexec)
    if (g) {
      (void)hipGraphExecDestroy(g);
      g = nullptr;
    }
}

void batch_release(ddcc_batch* b) {
  drop_graphs(b);
  void* ptrs[] = {b->f[0],   b->f[1], b->f0[0],    b->f0[1],    b->g[0],
                  b->g[1],   b->T[0], b->T[1],     b->hist,     b->psi,
                  b->wet,    b->staging, b->partial, b->bad, b->tiles,
                  b->insts,  b->kds, b->kfs};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  if (b->own_stream && b->stream) (void)hipStreamDestroy(b->stream);
}

// Tile list for tile height ty: instances in order, tiles row-major.
int build_tiles(ddcc_batch* b, int ty) {
  std::vector<BatchTile> tl;
  b->t0.assign(b->count, 0);
  b->t1.assign(b->count, 0);
  for (int i = 0; i < b->count; ++i) {
    b->t0[i] = (unsigned)tl.size();
    for (int y = 0; y < b->ny[i]; y += ty)
      for (int x = 0; x < b->nx[i]; x += 64) tl.push_back(BatchTile{i, x, y, 0});
    b->t1[i] = (unsigned)tl.size();
  }
  if (b->tiles) (void)hipFree(b->tiles);
  b->tiles = nullptr;
  BHIP(b, hipMalloc(&b->tiles, tl.size() * sizeof(BatchTile)), "hipMalloc tiles");
  BHIP(b, hipMemcpyAsync(b->tiles, tl.data(), tl.size() * sizeof(BatchTile),
                         hipMemcpyHostToDevice, b->stream),
       "copy tiles");
  BHIP(b, hipStreamSynchronize(b->stream), "sync");
  b->ntiles = (unsigned)tl.size();
  b->ty = ty;
  drop_graphs(b);
  return DDCC_OK;
}

template <class Pop, class S>
Bufs<Pop, S> batch_bufs(ddcc_batch* b, int mode) {
  Bufs<Pop, S> r{};
  const int a = b->cur, o = b->cur ^ 1;
  const int w = mode == MODE_INIT ? a : o;
  r.fA = static_cast<const Pop*>(b->f[a]);
  r.fB = static_cast<Pop*>(b->f[w]);
  r.f0A = b->f0[a];
  r.f0B = b->f0[w];
  r.gA = static_cast<const Pop*>(b->g[a]);
  r.gB = static_cast<Pop*>(b->g[w]);
  r.TA = static_cast<const S*>(b->T[a]);
  r.TB = static_cast<S*>(b->T[w]);
  r.hist = static_cast<S*>(b->hist);
  r.psi = static_cast<const S*>(b->psi);
  r.wet = static_cast<const S*>(b->wet);
  return r;
}

template <class Pop, class S, class R>
hipError_t batch_launch_as(ddcc_batch* b, const Coef<R>* k, int mode,
                           unsigned t0, unsigned nt, const double* inC,
                           const double* inU, const double* inP, double* oC,
                           double* oU, double* oP, long long out_n) {
  Bufs<Pop, S> r = batch_bufs<Pop, S>(b, mode);
  if (mode == MODE_STEP && b->stream_stores) {
    mode = MODE_STREAM;
    for (int nx : b->nx)
      if (!rows_on_lines(nx, sizeof(Pop))) mode = MODE_RAGGED;
  }
  r.inC = inC;
  r.inU = inU;
  r.inP = inP;
  r.outC = oC;
  r.outU = oU;
  r.outP = oP;
  r.out_n = out_n;
  return launch_2d_batch<Pop, S, R>(b->p.nphase, mode, b->kds, k, r,
                                    b->tiles + t0, b->insts, nt, b->ty,
                                    b->stream);
}

// Run `mode` over tiles [t0, t0 + nt).
hipError_t batch_launch(ddcc_batch* b, int mode, unsigned t0, unsigned nt,
                        const double* inC = nullptr,
                        const double* inU = nullptr, const double* inP = nullptr,
                        double* oC = nullptr, double* oU = nullptr,
                        double* oP = nullptr, long long out_n = 0) {
  switch (b->p.precision) {
    case DDCC_FP64:
      return batch_launch_as<double, double>(b, b->kds, mode, t0, nt, inC, inU,
                                             inP, oC, oU, oP, out_n);
    case DDCC_FP16:
      return batch_launch_as<_Float16, float>(b, b->kfs, mode, t0, nt, inC, inU,
                                              inP, oC, oU, oP, out_n);
    case DDCC_BF16:
      return batch_launch_as<__bf16, float>(b, b->kfs, mode, t0, nt, inC, inU,
                                            inP, oC, oU, oP, out_n);
    default:
      return batch_launch_as<float, float>(b, b->kfs, mode, t0, nt, inC, inU,
                                           inP, oC, oU, oP, out_n);
  }
}

// Copies instance i's planes [0, planes) between a host array laid out
// [plane][n_i] and batch-layout device memory [plane][ntot] at off_i.
int copy_planes(ddcc_batch* b, int i, void* dev, const void* host, int planes,
                size_t esz, hipMemcpyKind kind) {
  for (int q = 0; q < planes; ++q) {
    char* d = static_cast<char*>(dev) + ((size_t)q * b->ntot + b->off[i]) * esz;
    const char* h = static_cast<const char*>(host) + (size_t)q * b->n[i] * esz;
    hipError_t e = kind == hipMemcpyHostToDevice
                       ? hipMemcpyAsync(d, h, b->n[i] * esz, kind, b->stream)
                       : hipMemcpyAsync(const_cast<char*>(h), d, b->n[i] * esz,
                                        kind, b->stream);
    if (e != hipSuccess) return bhip(b, e, "plane copy");
  }
  return DDCC_OK;
}

int batch_check(ddcc_batch* b, int i) {
  if (!b) return DDCC_E_INVAL;
  if (i < 0 || i >= b->count) return bfail(b, DDCC_E_INVAL, "instance out of range");
  return DDCC_OK;
}

// One step of every instance.
int batch_step_direct(ddcc_batch* b) {
  hipError_t e = batch_launch(b, MODE_STEP, 0, b->ntiles);
  if (e != hipSuccess) return bhip(b, e, "batch step kernel");
  b->cur ^= 1;
  ++b->t;
  return DDCC_OK;
}

int batch_capture(ddcc_batch* b) {
  const int par = b->cur;
  hipGraph_t graph = nullptr;
  BHIP(b, hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal),
       "begin capture");
  hipError_t e = hipSuccess;
  for (int s = 0; s < b->graph_steps && e == hipSuccess; ++s) {
    e = batch_launch(b, MODE_STEP, 0, b->ntiles);
    b->cur ^= 1;
  }
  b->cur = par;
  hipError_t e2 = hipStreamEndCapture(b->stream, &graph);
  if (e != hipSuccess || e2 != hipSuccess) {
    if (graph) (void)hipGraphDestroy(graph);
    return bhip(b, e != hipSuccess ? e : e2, "graph capture");
  }
  e = hipGraphInstantiate(&b->gexec[par], graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) {
    b->gexec[par] = nullptr;
    return bhip(b, e, "graph instantiate");
  }
  return DDCC_OK;
}

}  // namespace

extern "C" {

int ddcc_batch_create(const ddcc_params* p, int count, const int* nx,
                      const int* ny, void* stream, ddcc_batch** out) {
  if (!out) return DDCC_E_INVAL;
  *out = nullptr;
  if (!p || !nx || !ny || count < 1) return DDCC_E_INVAL;
  if (p->dim != 2) return DDCC_E_UNSUPPORTED;
  long long ntot = 0;
  for (int i = 0; i < count; ++i) {
    if (nx[i] < 1 || ny[i] < 1) return DDCC_E_INVAL;
    ntot += (long long)nx[i] * ny[i];
  }
  if (ntot > (1LL << 29)) return DDCC_E_INVAL;
  ddcc_params q = *p;
  q.nx = nx[0];
  q.ny = ny[0];
  q.nz = 1;
  std::string msg;
  int rc = validate(&q, msg);
  if (rc != DDCC_OK) return rc;
  ddcc_batch* b = new (std::nothrow) ddcc_batch();
  if (!b) return DDCC_E_NOMEM;
  b->p = q;
  b->count = count;
  b->nx.assign(nx, nx + count);
  b->ny.assign(ny, ny + count);
  for (int i = 0; i < count; ++i) {
    b->n.push_back((long long)nx[i] * ny[i]);
    b->off.push_back(b->ntot);
    b->ntot += b->n.back();
  }
  b->geom_ok.assign(count, 0);
  b->fields_ok.assign(count, 0);
  b->esz = q.precision == DDCC_FP64 ? 8 : 4;
  b->pesz = q.precision == DDCC_FP64 ? 8 : (q.precision == DDCC_FP32 ? 4 : 2);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    delete b;
    return DDCC_E_HIP;
  }
  // A captured graph cannot use the legacy default stream.
  if (stream) {
    b->stream = static_cast<hipStream_t>(stream);
  } else {
    if (hipStreamCreate(&b->stream) != hipSuccess) {
      delete b;
      return DDCC_E_HIP;
    }
    b->own_stream = true;
  }
  // kernel constants: plane stride ntot; the box sizes come per instance
  ddcc_params qs = q;
  fill_coef<double>(qs, qs.nx, b->ntot, b->kd);
  fill_coef<float>(qs, qs.nx, b->ntot, b->kf);
  const int N = q.nphase;
  const size_t nt = (size_t)b->ntot;
  hipError_t e = hipSuccess;
  for (int a = 0; a < 2 && e == hipSuccess; ++a) {
    e = hipMalloc(&b->f[a], (size_t)N * (kBatchQ - 1) * nt * b->pesz);
    if (e == hipSuccess) e = hipMalloc(&b->f0[a], (size_t)N * nt * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&b->g[a], (size_t)kBatchQ * nt * b->pesz);
    if (e == hipSuccess) e = hipMalloc(&b->T[a], nt * b->esz);
  }
  if (e == hipSuccess) e = hipMalloc(&b->hist, (size_t)nhist_of(N) * nt * b->esz);
  b->stream_stores =
      step_bytes((size_t)N * (kBatchQ - 1) * nt * b->pesz +
                     (size_t)N * nt * sizeof(double) + (size_t)kBatchQ * nt * b->pesz,
                 nt * b->esz, (size_t)nhist_of(N) * nt * b->esz, 0) > kCacheBytes;
  if (e == hipSuccess) e = hipMalloc(&b->psi, nt * b->esz);
  if (e == hipSuccess) e = hipMalloc(&b->wet, (size_t)(N - 1) * nt * b->esz);
  if (e == hipSuccess)
    e = hipMalloc(&b->staging, (size_t)(N + 3) * nt * sizeof(double));
  long long mb = (ntot + 255) / 256;
  b->mass_blocks = (int)(mb > 1024 ? 1024 : mb);
  if (e == hipSuccess)
    e = hipMalloc(&b->partial, (size_t)b->mass_blocks * N * sizeof(double));
  if (e == hipSuccess) e = hipMalloc(&b->bad, (size_t)b->mass_blocks * sizeof(int));
  if (e == hipSuccess) {
    std::vector<BatchInst> ins(count);
    for (int i = 0; i < count; ++i) ins[i] = BatchInst{nx[i], ny[i], b->n[i], b->off[i]};
    e = hipMalloc(&b->insts, count * sizeof(BatchInst));
    if (e == hipSuccess)
      e = hipMemcpy(b->insts, ins.data(), count * sizeof(BatchInst),
                    hipMemcpyHostToDevice);
  }
  if (e == hipSuccess) {
    const std::vector<Coef<double>> vd(count, b->kd);
    const std::vector<Coef<float>> vf(count, b->kf);
    e = hipMalloc(&b->kds, count * sizeof(Coef<double>));
    if (e == hipSuccess) e = hipMalloc(&b->kfs, count * sizeof(Coef<float>));
    if (e == hipSuccess)
      e = hipMemcpy(b->kds, vd.data(), count * sizeof(Coef<double>),
                    hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = hipMemcpy(b->kfs, vf.data(), count * sizeof(Coef<float>),
                    hipMemcpyHostToDevice);
  }
  // 64 x 4 tiles for float64 as in single boxes (128 instances of 64^2 to 256^2:
  // 335 against 349 us per step with 64 x 8; 12 of 90 to 120 nodes a side 19.6
  // against 24.0), 64 x 8 for float
  if (e != hipSuccess ||
      build_tiles(b, q.precision == DDCC_FP64 ? 4 : 8) != DDCC_OK) {
    (void)hipGetLastError();  // see hip_fail
    batch_release(b);
    delete b;
    return e == hipErrorOutOfMemory ? DDCC_E_NOMEM : DDCC_E_HIP;
  }
  *out = b;
  return DDCC_OK;
}

int ddcc_batch_set_params(ddcc_batch* b, int i, const ddcc_params* p) {
  int rc = batch_check(b, i);
  if (rc) return rc;
  if (!p) return bfail(b, DDCC_E_INVAL, "params is NULL");
  if (p->dim != b->p.dim || p->nphase != b->p.nphase ||
      p->lattice_f != b->p.lattice_f || p->lattice_g != b->p.lattice_g ||
      p->precision != b->p.precision)
    return bfail(b, DDCC_E_INVAL,
                 "dim, nphase, lattices and precision must be the batch's");
  ddcc_params q = *p;
  q.nx = b->nx[i];
  q.ny = b->ny[i];
  q.nz = 1;
  std::string msg;
  rc = validate(&q, msg);
  if (rc != DDCC_OK) return bfail(b, rc, msg);
  Coef<double> kd;
  Coef<float> kf;
  fill_coef<double>(q, q.nx, b->ntot, kd);
  fill_coef<float>(q, q.nx, b->ntot, kf);
  // the tables are read by kernels on the batch stream
  if (hipStreamSynchronize(b->stream) != hipSuccess ||
      hipMemcpy(b->kds + i, &kd, sizeof(kd), hipMemcpyHostToDevice) !=
          hipSuccess ||
      hipMemcpy(b->kfs + i, &kf, sizeof(kf), hipMemcpyHostToDevice) !=
          hipSuccess)
    return bfail(b, DDCC_E_HIP, "copy parameters");
  return DDCC_OK;
}

int ddcc_batch_init_geometry(ddcc_batch* b, int i, const double* psi,
                             const double* ct) {
  int rc = batch_check(b, i);
  if (rc) return rc;
  if (!psi) return bfail(b, DDCC_E_INVAL, "psi is NULL");
  const size_t n = (size_t)b->n[i];
  const int N = b->p.nphase;
  for (size_t k = 0; k < n; ++k)
    if (!(psi[k] >= 0.0 && psi[k] <= 1.0))
      return bfail(b, DDCC_E_INVAL, "psi outside [0, 1]");
  if (ct)
    for (size_t k = 0; k < (size_t)(N - 1) * n; ++k)
      if (!(ct[k] >= -1.0 && ct[k] <= 1.0))
        return bfail(b, DDCC_E_INVAL, "cos theta outside [-1, 1]");
  // psi and the wetting weights of the instance, computed on the device
  const size_t nc = ct ? (size_t)(N - 1) * n : 0;
  double* d = nullptr;
  BHIP(b, hipMalloc(&d, (n + nc) * sizeof(double)), "hipMalloc geometry");
  hipError_t e = hipMemcpyAsync(d, psi, n * sizeof(double),
                                hipMemcpyHostToDevice, b->stream);
  if (e == hipSuccess && nc)
    e = hipMemcpyAsync(d + n, ct, nc * sizeof(double), hipMemcpyHostToDevice,
                       b->stream);
  if (e == hipSuccess)
    e = b->p.precision == DDCC_FP64
            ? launch_wet_field<double>(d, nc ? d + n : nullptr, 1, N - 1,
                                       b->nx[i], b->ny[i], 1, b->nx[i],
                                       static_cast<double*>(b->psi),
                                       static_cast<double*>(b->wet), b->ntot,
                                       b->off[i], b->stream)
            : launch_wet_field<float>(d, nc ? d + n : nullptr, 1, N - 1,
                                      b->nx[i], b->ny[i], 1, b->nx[i],
                                      static_cast<float*>(b->psi),
                                      static_cast<float*>(b->wet), b->ntot,
                                      b->off[i], b->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  (void)hipFree(d);
  if (e != hipSuccess) return bhip(b, e, "batch geometry");
  b->geom_ok[i] = 1;
  b->fields_ok[i] = 0;
  return DDCC_OK;
}

int ddcc_batch_init_fields(ddcc_batch* b, int i, const double* C,
                           const double* u, const double* P) {
  int rc = batch_check(b, i);
  if (rc) return rc;
  if (!b->geom_ok[i]) return bfail(b, DDCC_E_STATE, "init_geometry first");
  if (!C) return bfail(b, DDCC_E_INVAL, "C is NULL");
  const int N = b->p.nphase;
  const size_t n = (size_t)b->n[i];
  if (!all_finite(C, N * n) || (u && !all_finite(u, 2 * n)) ||
      (P && !all_finite(P, n)))
    return bfail(b, DDCC_E_INVAL, "non-finite initial field");
  double* sC = b->staging;
  double* sU = sC + (size_t)N * b->ntot;
  double* sP = sU + 2 * (size_t)b->ntot;
  rc = copy_planes(b, i, sC, C, N, sizeof(double), hipMemcpyHostToDevice);
  if (!rc && u) rc = copy_planes(b, i, sU, u, 2, sizeof(double), hipMemcpyHostToDevice);
  if (!rc && P) rc = copy_planes(b, i, sP, P, 1, sizeof(double), hipMemcpyHostToDevice);
  if (rc) return rc;
  // initialisation writes the populations of the current level in place
  hipError_t e = batch_launch(b, MODE_INIT, b->t0[i], b->t1[i] - b->t0[i],
                              sC, u ? sU : nullptr, P ? sP : nullptr);
  if (e != hipSuccess) return bhip(b, e, "batch init kernel");
  BHIP(b, hipStreamSynchronize(b->stream), "sync");
  b->fields_ok[i] = 1;
  return DDCC_OK;
}

int ddcc_batch_step(ddcc_batch* b, int64_t nsteps) {
  if (!b) return DDCC_E_INVAL;
  if (nsteps < 0) return bfail(b, DDCC_E_INVAL, "nsteps < 0");
  for (int i = 0; i < b->count; ++i)
    if (!b->fields_ok[i])
      return bfail(b, DDCC_E_STATE, "every instance needs init_fields first");
  int64_t left = nsteps;
  if (b->graph_steps > 0) {
    while (left >= b->graph_steps) {
      if (!b->gexec[b->cur]) {
        int rc = batch_capture(b);
        if (rc) return rc;
      }
      BHIP(b, hipGraphLaunch(b->gexec[b->cur], b->stream), "graph launch");
      // an even number of steps leaves the level parity unchanged
      b->t += b->graph_steps;
      left -= b->graph_steps;
    }
  }
  for (; left > 0; --left) {
    int rc = batch_step_direct(b);
    if (rc) return rc;
  }
  return DDCC_OK;
}

int ddcc_batch_read_moments(ddcc_batch* b, int i, double* C, double* u,
                            double* P) {
  int rc = batch_check(b, i);
  if (rc) return rc;
  if (!b->fields_ok[i]) return bfail(b, DDCC_E_STATE, "init_fields first");
  const int N = b->p.nphase;
  // the instance's planes one after another, so that each field is one copy
  const size_t n = (size_t)b->n[i];
  double* sC = b->staging;
  double* sU = sC + (size_t)N * n;
  double* sP = sU + 2 * n;
  const long long o = b->off[i];  // the kernel's node index starts there
  hipError_t e = batch_launch(b, MODE_MOMENTS, b->t0[i], b->t1[i] - b->t0[i],
                              nullptr, nullptr, nullptr, sC - o, sU - o, sP - o,
                              (long long)n);
  if (e != hipSuccess) return bhip(b, e, "batch moments kernel");
  const struct {
    double* host;
    const double* dev;
    size_t planes;
  } parts[3] = {{C, sC, (size_t)N}, {u, sU, 2}, {P, sP, 1}};
  for (const auto& q : parts)
    if (q.host)
      BHIP(b, hipMemcpyAsync(q.host, q.dev, q.planes * n * sizeof(double),
                             hipMemcpyDeviceToHost, b->stream),
           "copy moments");
  BHIP(b, hipStreamSynchronize(b->stream), "sync");
  return DDCC_OK;
}

int ddcc_batch_mass(ddcc_batch* b, int i, double* mass) {
  int rc = batch_check(b, i);
  if (rc) return rc;
  if (!mass) return bfail(b, DDCC_E_INVAL, "mass is NULL");
  if (!b->fields_ok[i]) return bfail(b, DDCC_E_STATE, "init_fields first");
  const int N = b->p.nphase;
  const long long o = b->off[i];
  const double* f0 = b->f0[b->cur] + o;
  hipError_t e;
  switch (b->p.precision) {
    case DDCC_FP64:
      e = launch_mass(f0, static_cast<const double*>(b->f[b->cur]) + o, N,
                      kBatchQ, b->n[i], b->ntot, b->partial, b->bad,
                      b->mass_blocks, b->stream);
      break;
    case DDCC_FP16:
      e = launch_mass(f0, static_cast<const _Float16*>(b->f[b->cur]) + o, N,
                      kBatchQ, b->n[i], b->ntot, b->partial, b->bad,
                      b->mass_blocks, b->stream);
      break;
    case DDCC_BF16:
      e = launch_mass(f0, static_cast<const __bf16*>(b->f[b->cur]) + o, N,
                      kBatchQ, b->n[i], b->ntot, b->partial, b->bad,
                      b->mass_blocks, b->stream);
      break;
    default:
      e = launch_mass(f0, static_cast<const float*>(b->f[b->cur]) + o, N,
                      kBatchQ, b->n[i], b->ntot, b->partial, b->bad,
                      b->mass_blocks, b->stream);
  }
  if (e != hipSuccess) return bhip(b, e, "mass kernel");
  std::vector<double> part((size_t)b->mass_blocks * N);
  std::vector<int> bad(b->mass_blocks);
  BHIP(b, hipMemcpyAsync(part.data(), b->partial, part.size() * sizeof(double),
                         hipMemcpyDeviceToHost, b->stream),
       "copy partials");
  BHIP(b, hipMemcpyAsync(bad.data(), b->bad, bad.size() * sizeof(int),
                         hipMemcpyDeviceToHost, b->stream),
       "copy flags");
  BHIP(b, hipStreamSynchronize(b->stream), "sync");
  for (int k = 0; k < N; ++k) {
    double s = 0.0;
    for (int q = 0; q < b->mass_blocks; ++q) s += part[(size_t)q * N + k];
    mass[k] = s;
  }
  for (int q = 0; q < b->mass_blocks; ++q)
    if (bad[q]) return bfail(b, DDCC_E_NONFINITE, "non-finite population");
  return DDCC_OK;
}

int ddcc_batch_set_tile(ddcc_batch* b, int ty) {
  if (!b) return DDCC_E_INVAL;
  if (ty != 4 && ty != 8 && ty != 16)
    return bfail(b, DDCC_E_INVAL, "batch tile height must be 4, 8 or 16");
  return build_tiles(b, ty);
}

int ddcc_batch_set_graph(ddcc_batch* b, int steps_per_graph) {
  if (!b) return DDCC_E_INVAL;
  if (steps_per_graph < 0 || steps_per_graph > kMaxGraphSteps ||
      steps_per_graph % 2 != 0)
    return bfail(b, DDCC_E_INVAL,
                 "steps per graph must be even and in [0, 1024]");
  drop_graphs(b);
  b->graph_steps = steps_per_graph;
  return DDCC_OK;
}

int ddcc_batch_autotune(ddcc_batch* b, int steps, int* ty_out) {
  if (!b) return DDCC_E_INVAL;
  if (steps < 1) return bfail(b, DDCC_E_INVAL, "steps < 1");
  for (int i = 0; i < b->count; ++i)
    if (!b->fields_ok[i])
      return bfail(b, DDCC_E_STATE, "every instance needs init_fields first");
  // The trial steps change the state: keep a copy of the current level.
  const int N = b->p.nphase;
  const size_t nt = (size_t)b->ntot;
  const size_t sizes[5] = {(size_t)N * (kBatchQ - 1) * nt * b->pesz,
                           (size_t)N * nt * sizeof(double),
                           (size_t)kBatchQ * nt * b->pesz, nt * b->esz,
                           (size_t)nhist_of(N) * nt * b->esz};
  const int cur0 = b->cur;
  void* src[5] = {b->f[cur0], b->f0[cur0], b->g[cur0], b->T[cur0], b->hist};
  void* keep[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  hipError_t e = hipSuccess;
  for (int q = 0; q < 5 && e == hipSuccess; ++q) {
    e = hipMalloc(&keep[q], sizes[q]);
    if (e == hipSuccess)
      e = hipMemcpyAsync(keep[q], src[q], sizes[q], hipMemcpyDeviceToDevice,
                         b->stream);
  }
  const int cands[3] = {4, 8, 16};
  float best_ms = 0;
  int best = b->ty;
  hipEvent_t t0 = nullptr, t1 = nullptr;
  if (e == hipSuccess) e = hipEventCreate(&t0);
  if (e == hipSuccess) e = hipEventCreate(&t1);
  const int64_t tsave = b->t;
  for (int c = 0; c < 3 && e == hipSuccess; ++c) {
    if (build_tiles(b, cands[c]) != DDCC_OK) {
      e = hipErrorUnknown;
      break;
    }
    for (int w = 0; w < 2 && e == hipSuccess; ++w)
      if (batch_step_direct(b) != DDCC_OK) e = hipErrorUnknown;
    if (e == hipSuccess) e = hipEventRecord(t0, b->stream);
    for (int s = 0; s < steps && e == hipSuccess; ++s)
      if (batch_step_direct(b) != DDCC_OK) e = hipErrorUnknown;
    if (e == hipSuccess) e = hipEventRecord(t1, b->stream);
    if (e == hipSuccess) e = hipEventSynchronize(t1);
    float ms = 0;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, t0, t1);
    if (e == hipSuccess && (c == 0 || ms < best_ms)) {
      best_ms = ms;
      best = cands[c];
    }
  }
  // restore the level the trials started from
  b->cur = cur0;
  b->t = tsave;
  for (int q = 0; q < 5; ++q)
    if (keep[q]) {
      if (e == hipSuccess)
        e = hipMemcpyAsync(src[q], keep[q], sizes[q], hipMemcpyDeviceToDevice,
                           b->stream);
    }
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  for (int q = 0; q < 5; ++q)
    if (keep[q]) (void)hipFree(keep[q]);
  if (t0) (void)hipEventDestroy(t0);
  if (t1) (void)hipEventDestroy(t1);
  if (e != hipSuccess) return bhip(b, e, "autotune");
  int rc = build_tiles(b, best);
  if (rc) return rc;
  if (ty_out) *ty_out = best;
  return DDCC_OK;
}

int ddcc_batch_sync(ddcc_batch* b) {
  if (!b) return DDCC_E_INVAL;
  BHIP(b, hipStreamSynchronize(b->stream), "sync");
  return DDCC_OK;
}

int64_t ddcc_batch_time(const ddcc_batch* b) { return b ? b->t : -1; }

const char* ddcc_batch_last_error(const ddcc_batch* b) {
  return b ? b->err.c_str() : "NULL batch";
}

void ddcc_batch_destroy(ddcc_batch* b) {
  if (!b) return;
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  batch_release(b);
  delete b;
}

}  // extern "C"
