// Host side of the library: contexts, launches, graphs, tile tuning, batch
// runs and the C ABI declared in include/lbm.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "lbm.h"
#include "lbm_internal.h"
#include "lbm_kernels.hpp"

namespace lbm {
namespace {

constexpr int kEXh[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int kEYh[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
const double kWh[9] = {4.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0,
                       1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};
constexpr size_t kAlign = 256;
constexpr int kMassBlocks = 1024;
constexpr unsigned long long kNoDiv = ~0ull;

#define HIPCHK(x)                        \
  do {                                   \
    if ((x) != hipSuccess) return LBM_EHIP; \
  } while (0)

// Launch shape of the step kernels: waves per block (one-step kernels: a strip of
// 64*nw columns; multi-step kernels: strip class, see pipe_nw), rows per block (0 =
// balanced schedule over the resident grid), the row prefetch depth of the one-step
// kernels (1 or 2) and the time steps per launch.
struct Tile {
  int nw, L, pf;
  int ts = 1;
};

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
int esize_of(int prec) { return prec == LBM_PREC_F64 ? 8 : prec == LBM_PREC_F16DEV ? 2 : 4; }
using layout::elems_of;
using layout::pitch_of;
using layout::plane_of;
using layout::rs_of;

int validate(const lbm_params& p) {
  if (p.nx < 3 || p.ny < 3) return LBM_EINVAL;
  if ((int64_t)p.nx * p.ny >= (1ll << 31)) return LBM_EINVAL;
  if (!(p.tau > 0.5) || !std::isfinite(p.tau)) return LBM_EINVAL;
  if (!(p.G != 0.0) || !std::isfinite(p.G)) return LBM_EINVAL;
  if (p.eos != LBM_EOS_CS && p.eos != LBM_EOS_PR) return LBM_EINVAL;
  if (p.scheme < LBM_SCHEME_SHANCHEN || p.scheme > LBM_SCHEME_LADD) return LBM_EINVAL;
  if (p.precision < LBM_PREC_F64 || p.precision > LBM_PREC_F32DEV_F64) return LBM_EINVAL;
  if (!(p.a > 0) || !(p.b > 0) || !(p.R > 0) || !(p.T > 0)) return LBM_EINVAL;
  if (!std::isfinite(p.sigma)) return LBM_EINVAL;
  return LBM_OK;
}

double host_psi2(const EosConst& k, double rho) { return (pressure(k, rho) - rho / 3.0) * k.two_over_G; }

// Host equilibrium, Eq. (2) with c_s^2 = 1/3.
void host_feq(double rho, double ux, double uy, double* f) {
  const double usq = ux * ux + uy * uy;
  for (int a = 0; a < 9; ++a) {
    const double eu = kEXh[a] * ux + kEYh[a] * uy;
    f[a] = kWh[a] * rho * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * usq);
  }
}

// Fill the device-side constants of one lattice.
RunDev make_rundev(const lbm_params& p, const EosConst& k, double rho_ref, int64_t off, int run) {
  RunDev d{};
  d.nx = p.nx;
  d.ny = p.ny;
  d.pitch = pitch_of(p.nx);
  d.eos = p.eos;
  d.plane = plane_of(p.nx);
  d.rs = rs_of(p.nx);
  d.elems = elems_of(p.nx, p.ny);
  d.off = off;
  d.RT = k.RT;
  d.c1 = k.c1;
  d.c2 = k.c2;
  d.two_over_G = k.two_over_G;
  d.mG = -p.G;
  d.inv_tau = 1.0 / p.tau;
  double Be = 0.0;
  switch (p.scheme) {
    case LBM_SCHEME_SHANCHEN:  // Eqs. (9)-(10): u_eq = u + tau F/rho, no forcing term
      d.c_eq = p.tau;
      d.c_f = 0.0;
      d.sig = 0.0;
      Be = d.Ce = 0.0;
      break;
    case LBM_SCHEME_EDM:  // Eq. (11) = Eq. (16): B_e = C_e = 1, velocity u + F/(2 rho)
      d.c_eq = 0.0;
      d.c_f = 0.5;
      d.sig = 0.0;
      Be = d.Ce = 1.0;
      break;
    case LBM_SCHEME_EDM_MODIFIED:  // Sec. III.C: EDM with C_e = 1/tau
      d.c_eq = 0.0;
      d.c_f = 0.5;
      d.sig = 0.0;
      Be = 1.0;
      d.Ce = 1.0 / p.tau;
      break;
    case LBM_SCHEME_LADD:  // Table I: u in the equilibrium and in F_a, B_e = C_e = 1
      d.c_eq = 0.0;
      d.c_f = 0.0;
      d.sig = 0.0;
      Be = d.Ce = 1.0;
      break;
    default:  // Eq. (31): u_eq = v, B_e = C_e = 1 - 1/(2 tau), v' = v + sigma F/((tau - 1/2) psi^2)
      d.c_eq = 0.5;
      d.c_f = 0.5;
      d.sig = p.sigma / (p.tau - 0.5);
      Be = d.Ce = 1.0 - 0.5 / p.tau;
      break;
  }
  d.c_d = d.c_f - d.c_eq;
  d.om_2 = d.inv_tau / 2.0;
  d.om_3 = d.inv_tau / 3.0;
  d.Be_3 = Be / 3.0;
  d.wCe0 = 4.0 / 9.0 * d.Ce;
  d.wCe1 = 1.0 / 9.0 * d.Ce;
  d.wCe2 = 1.0 / 36.0 * d.Ce;
  d.wBe3_1 = 3.0 / 9.0 * Be;
  d.wBe3_2 = 3.0 / 36.0 * Be;
  d.om_w0 = 4.0 / 9.0 * d.inv_tau;
  d.om_w1 = 1.0 / 9.0 * d.inv_tau;
  d.om_w2 = 1.0 / 36.0 * d.inv_tau;
  d.om_3w1 = 3.0 / 9.0 * d.inv_tau;
  d.om_3w2 = 3.0 / 36.0 * d.inv_tau;
  d.om1 = 1.0 - d.inv_tau;
  d.rho_ref = rho_ref;
  d.run = run;
  d.mrt = 0;
  return d;
}

// Switch a lattice's constants to the MRT collision with energy, energy-square
// and energy-flux rates r[0..2] (the density, momentum and stress moments relax
// at 1/tau): sigma / (1/s - 1/2) of the improved scheme per moment.
void set_mrt(RunDev& d, const lbm_params& p, const double* r) {
  auto h = [](double s) { return 1.0 - 0.5 * s; };
  const double n = d.inv_tau;
  d.mrt = 1;
  d.m = MrtDev{-r[0] / 36.0, h(r[0]) / 6.0,  p.sigma / (1.0 / r[0] - 0.5),
               -r[1] / 36.0, -h(r[1]) / 6.0, p.sigma / (1.0 / r[1] - 0.5),
               r[2] / 6.0,   (1.0 + h(r[2])) / 6.0, -r[2] / 12.0, 1.0 / 6.0 - h(r[2]) / 12.0,
               -n / 4.0,     h(n) / 2.0,     h(n) / 4.0};
}

// Encode FP64 populations into the storage buffer (layout::encode): FP64 as
// is, deviations f - w rho_ref rounded to FP32 (and then to FP16).
template <typename S>
void encode_buffer(const lbm_params& p, double rref, const double* f, std::vector<char>& out) {
  out.assign(elems_of(p.nx, p.ny) * sizeof(S), 0);
  S* b = reinterpret_cast<S*>(out.data());
  layout::encode(p.nx, p.ny, f, b, [&](int a, double v) -> S {
    if constexpr (std::is_same<S, double>::value)
      return v;
    else if constexpr (std::is_same<S, float>::value)
      return (float)(v - kWh[a] * rref);
    else  // RNE to FP32, then RNE to FP16
      return __float2half_rn((float)(v - kWh[a] * rref));
  });
}

// Decode the storage buffer to FP64 populations: f = s + (w rho_ref), two
// separately rounded operations (as the device decoder of the mass does).
template <typename S>
void decode_buffer(const lbm_params& p, double rref, const char* raw, double* f) {
  const S* b = reinterpret_cast<const S*>(raw);
  layout::decode(p.nx, p.ny, b, f, [&](int a, S v) -> double {
    if constexpr (std::is_same<S, double>::value) {
      return v;
    } else {
      volatile double wr = kWh[a] * rref;  // keep the two roundings separate
      if constexpr (std::is_same<S, float>::value)
        return (double)v + wr;
      else
        return (double)__half2float(v) + wr;
    }
  });
}

void encode_any(int prec, const lbm_params& p, double rref, const double* f, std::vector<char>& o) {
  if (prec == LBM_PREC_F64) encode_buffer<double>(p, rref, f, o);
  else if (prec == LBM_PREC_F16DEV) encode_buffer<__half>(p, rref, f, o);
  else encode_buffer<float>(p, rref, f, o);
}
void decode_any(int prec, const lbm_params& p, double rref, const char* raw, double* f) {
  if (prec == LBM_PREC_F64) decode_buffer<double>(p, rref, raw, f);
  else if (prec == LBM_PREC_F16DEV) decode_buffer<__half>(p, rref, raw, f);
  else decode_buffer<float>(p, rref, raw, f);
}

// ---- launches ---------------------------------------------------------------

// CUs, and resident blocks per CU, for one kernel (cached per kernel).
struct Residency {
  int ncu, per_cu;
};
Residency residency(const void* fn, int threads) {
  static std::mutex mu;
  static std::map<const void*, Residency> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find(fn);
  if (it != cache.end()) return it->second;
  int dev = 0, ncu = 256, occ = 1;
  if (hipGetDevice(&dev) == hipSuccess) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) ncu = prop.multiProcessorCount;
  }
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, 0) != hipSuccess || occ < 1)
    occ = 1;
  return cache[fn] = Residency{ncu, occ};
}
int resident_blocks(const void* fn, int threads) {
  const Residency r = residency(fn, threads);
  return r.ncu * r.per_cu;
}

template <typename S, int NW, int PF, bool MRT>
hipError_t launch_step_t(const void* src, void* dst, const RunDev& d, int L,
                         const unsigned long long* base, unsigned long long local,
                         unsigned long long* flag, hipStream_t st) {
  const int SW = 64 * NW;
  const int nstrips = (d.nx + SW - 1) / SW;
  if (!layout::launchable(layout::chunks(nstrips, d.ny, L), SW)) L = 0;
  int grid;
  if (L > 0) {
    grid = (int)layout::chunks(nstrips, d.ny, L);
  } else {  // balanced: resident capacity, at least 8 rows per block
    const int64_t rows = (int64_t)nstrips * d.ny;
    grid = resident_blocks((const void*)k_step<S, NW, PF, MRT>, SW);
    grid = (int)std::max<int64_t>(1, std::min<int64_t>(grid, rows / 8));
  }
  using E = typename Store<S>::E;
  hipLaunchKernelGGL((k_step<S, NW, PF, MRT>), dim3(grid), dim3(SW), 0, st, static_cast<const E*>(src),
                     static_cast<E*>(dst), d, L, nstrips, base, local, flag);
  return hipGetLastError();
}

template <typename S, bool MRT = false>
hipError_t launch_step_s(const Tile& t, const void* src, void* dst, const RunDev& d,
                         const unsigned long long* base, unsigned long long local,
                         unsigned long long* flag, hipStream_t st) {
  switch (t.nw * 10 + t.pf) {
    case 11: return launch_step_t<S, 1, 1, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 12: return launch_step_t<S, 1, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 21: return launch_step_t<S, 2, 1, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 22: return launch_step_t<S, 2, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 41: return launch_step_t<S, 4, 1, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 42: return launch_step_t<S, 4, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 81: return launch_step_t<S, 8, 1, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 82: return launch_step_t<S, 8, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
    case 161: return launch_step_t<S, 16, 1, MRT>(src, dst, d, t.L, base, local, flag, st);
    default: return launch_step_t<S, 16, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
  }
}

// Strips of a multi-step launch: at most W - 2H columns after their edges are aligned
// down to A columns (one strip needs no alignment).
template <typename S, int NW, int TS> int pipe_strips(int nx) {
  constexpr int M = 64 * NW - 2 * (2 * TS - 1), A = StripAlign<S>::value;
  return nx <= M ? 1 : (nx + M - A) / (M - A + 1);
}

template <typename S, int NW, int TS, bool MRT>
hipError_t launch_pipe_t(const void* src, void* dst, const RunDev& d, int L,
                         const unsigned long long* base, unsigned long long local,
                         unsigned long long* flag, hipStream_t st) {
  const int threads = 64 * NW * TS;
  const int nstrips = pipe_strips<S, NW, TS>(d.nx);
  if (!layout::launchable(layout::chunks(nstrips, d.ny, L), threads)) L = 0;
  int grid;
  if (L > 0) {
    grid = (int)layout::chunks(nstrips, d.ny, L);
  } else {
    // A second block on a CU halves the rows of a share but not its fill, so it pays only
    // while shares keep nearly a fill's rows (FP32, 128-column strips, us per step with one
    // and two blocks per CU: 22 rows against 11 8.8 and 10.0, 36 against 18 11.9 and 11.7,
    // 55 against 27 15.9 and 15.1).
    const int64_t rows = (int64_t)nstrips * d.ny;
    const Residency r = residency((const void*)k_pipe<S, NW, TS, MRT>, threads);
    const int64_t least = std::max(8, (pipe_fill(TS) + pipe_drain_rows(TS)) * 17 / 20);
    const int64_t k = std::max<int64_t>(1, std::min<int64_t>(r.per_cu, rows / (r.ncu * least)));
    grid = (int)std::max<int64_t>(1, std::min<int64_t>(r.ncu * k, rows / 8));
  }
  using E = typename Store<S>::E;
  hipLaunchKernelGGL((k_pipe<S, NW, TS, MRT>), dim3(grid), dim3(threads), 0, st,
                     static_cast<const E*>(src), static_cast<E*>(dst), d, L, nstrips, base, local, flag);
  return hipGetLastError();
}

// Storage types with three steps per launch as a tile: those with FP64 collision
// arithmetic.
bool has_step3(int prec) { return prec == LBM_PREC_F64 || prec == LBM_PREC_F32DEV_F64; }

template <typename S, int RX, int RY, int TS, bool MRT>
hipError_t launch_patch_t(const void* src, void* dst, const RunDev& d, const unsigned long long* base,
                          unsigned long long local, unsigned long long* flag, hipStream_t st) {
  static_assert(RX == RY && RX == layout::patch_side(TS), "layout's patch");
  const int ntx = layout::patches_across(d.nx, TS);
  const int64_t grid = layout::patches(d.nx, d.ny, TS);
  using E = typename Store<S>::E;
  hipLaunchKernelGGL((k_patch<S, RX, RY, TS, MRT>), dim3((unsigned)grid), dim3((RX * RY + 63) / 64 * 64), 0, st,
                     static_cast<const E*>(src), static_cast<E*>(dst), d, ntx, base, local, flag);
  return hipGetLastError();
}

template <typename S, bool MRT = false>
hipError_t launch_pipe_s(const Tile& t, const void* src, void* dst, const RunDev& d,
                         const unsigned long long* base, unsigned long long local,
                         unsigned long long* flag, hipStream_t st) {
  constexpr int NW = pipe_nw<S>(4);
  if (t.nw == 1) {  // patches (see k_patch)
    if (t.ts == 2) return launch_patch_t<S, 32, 32, 2, MRT>(src, dst, d, base, local, flag, st);
    if (t.ts == 3) return launch_patch_t<S, 32, 32, 3, MRT>(src, dst, d, base, local, flag, st);
    return launch_patch_t<S, 22, 22, 4, MRT>(src, dst, d, base, local, flag, st);
  }
  if (t.ts == 2) {
    // FP64 arithmetic: two steps leave room in a CU for one block with twice the columns
    // instead of two blocks; fewer columns are recomputed and fewer lines read twice.  Not
    // where the wide strips leave a quarter more lanes idle.  us per launch of two steps,
    // three waves per step and six: FP64 4096 x 4096 526 and 501, 1024 x 1024 49 and 43.5,
    // 777 x 643 33 and 27.6, 400 x 400 16.7 and 21; FP32 storage 4096 x 4096 378 and 302,
    // 1500 x 1001 49 and 38.  (FP32 arithmetic, four and eight: 304 and 301, 27 and 30.)
    if constexpr (std::is_same<typename Store<S>::R, double>::value)
      if (4 * 6 * pipe_strips<S, 6, 2>(d.nx) <= 5 * NW * pipe_strips<S, NW, 2>(d.nx))
        return launch_pipe_t<S, 6, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
    return launch_pipe_t<S, NW, 2, MRT>(src, dst, d, t.L, base, local, flag, st);
  }
  if (t.ts == 4)
    return t.nw == 2 ? launch_pipe_t<S, 2, 4, MRT>(src, dst, d, t.L, base, local, flag, st)
                     : launch_pipe_t<S, NW, 4, MRT>(src, dst, d, t.L, base, local, flag, st);
  if constexpr (std::is_same<typename Store<S>::R, double>::value)
    if (t.ts == 3) return launch_pipe_t<S, NW, 3, MRT>(src, dst, d, t.L, base, local, flag, st);
  return hipErrorInvalidValue;
}

// One launch of the tile: t.ts time steps from src into dst.
hipError_t launch_step(int prec, const Tile& t, const void* src, void* dst, const RunDev& d,
                       const unsigned long long* base, unsigned long long local,
                       unsigned long long* flag, hipStream_t st) {
  if (d.mrt) {  // FP64 or FP32 deviation storage (checked by lbm_set_mrt)
    if (t.ts > 1)
      return prec == LBM_PREC_F64 ? launch_pipe_s<double, true>(t, src, dst, d, base, local, flag, st)
                                  : launch_pipe_s<float, true>(t, src, dst, d, base, local, flag, st);
    if (prec == LBM_PREC_F64) return launch_step_s<double, true>(t, src, dst, d, base, local, flag, st);
    return launch_step_s<float, true>(t, src, dst, d, base, local, flag, st);
  }
  if (t.ts > 1) {
    if (prec == LBM_PREC_F64) return launch_pipe_s<double>(t, src, dst, d, base, local, flag, st);
    if (prec == LBM_PREC_F32DEV) return launch_pipe_s<float>(t, src, dst, d, base, local, flag, st);
    if (prec == LBM_PREC_F32DEV_F64)
      return launch_pipe_s<f32s_f64a>(t, src, dst, d, base, local, flag, st);
    return launch_pipe_s<__half>(t, src, dst, d, base, local, flag, st);
  }
  if (prec == LBM_PREC_F64) return launch_step_s<double>(t, src, dst, d, base, local, flag, st);
  if (prec == LBM_PREC_F32DEV) return launch_step_s<float>(t, src, dst, d, base, local, flag, st);
  if (prec == LBM_PREC_F32DEV_F64) return launch_step_s<f32s_f64a>(t, src, dst, d, base, local, flag, st);
  return launch_step_s<__half>(t, src, dst, d, base, local, flag, st);
}

// A batch launch.  grid 0: only report the resident blocks of the tile's kernel.
struct BatchArgs {
  const void* src;
  void* dst;
  const RunDev* runs;
  const Item* items;
  int nitems, total, grid;
  const unsigned long long* base;
  unsigned long long local;
  unsigned long long* flags;
  hipStream_t st;
  int* resident;
};

// Grid of a batch schedule with `resident` blocks of its kernel: item lists take at most
// one block per item; the balanced schedule (total > 0 rows) at least 8 rows per block.
constexpr int kMaxBatchGrid = 8192;  // 256 CUs of 32 waves
int batch_grid(int resident, int nitems, int total) {
  return std::max(1, std::min(std::min(resident, kMaxBatchGrid), total > 0 ? total / 8 : nitems));
}

template <typename S, class Kernel>
hipError_t launch_batch_k(Kernel k, int threads, const BatchArgs& a) {
  if (a.resident) {
    *a.resident = resident_blocks((const void*)k, threads);
    return hipSuccess;
  }
  using E = typename Store<S>::E;
  hipLaunchKernelGGL(k, dim3(a.grid), dim3(threads), 0, a.st, static_cast<const E*>(a.src),
                     static_cast<E*>(a.dst), a.runs, a.items, a.nitems, a.total, a.base, a.local, a.flags);
  return hipGetLastError();
}

template <typename S, bool MRT = false>
hipError_t launch_batch_s(const Tile& t, const BatchArgs& a) {
  switch (t.nw * 10 + t.pf) {
    case 11: return launch_batch_k<S>(k_batch_step<S, 1, 1, MRT>, 64, a);
    case 12: return launch_batch_k<S>(k_batch_step<S, 1, 2, MRT>, 64, a);
    case 21: return launch_batch_k<S>(k_batch_step<S, 2, 1, MRT>, 128, a);
    case 22: return launch_batch_k<S>(k_batch_step<S, 2, 2, MRT>, 128, a);
    case 41: return launch_batch_k<S>(k_batch_step<S, 4, 1, MRT>, 256, a);
    case 42: return launch_batch_k<S>(k_batch_step<S, 4, 2, MRT>, 256, a);
    case 81: return launch_batch_k<S>(k_batch_step<S, 8, 1, MRT>, 512, a);
    default: return launch_batch_k<S>(k_batch_step<S, 8, 2, MRT>, 512, a);
  }
}

template <typename S, bool MRT = false>
hipError_t launch_batch_pipe_s(const Tile& t, const BatchArgs& a) {
  constexpr int NW = pipe_nw<S>(4);
  if (t.ts == 4)
    return t.nw == 2 ? launch_batch_k<S>(k_batch_pipe<S, 2, 4, MRT>, 512, a)
                     : launch_batch_k<S>(k_batch_pipe<S, NW, 4, MRT>, 256 * NW, a);
  if (t.ts == 2)
    return t.nw == 2 ? launch_batch_k<S>(k_batch_pipe<S, 2, 2, MRT>, 256, a)
                     : launch_batch_k<S>(k_batch_pipe<S, NW, 2, MRT>, 128 * NW, a);
  return hipErrorInvalidValue;
}

// One launch of the batch tile: t.ts time steps of every active run;
// mrt: the runs' descriptors carry the MRT collision (FP64 or FP32 deviation
// storage, checked by lbm_batch_set_mrt).
hipError_t launch_batch(int prec, bool mrt, const Tile& t, const BatchArgs& a) {
  if (mrt) {
    if (t.ts > 1)
      return prec == LBM_PREC_F64 ? launch_batch_pipe_s<double, true>(t, a) : launch_batch_pipe_s<float, true>(t, a);
    return prec == LBM_PREC_F64 ? launch_batch_s<double, true>(t, a) : launch_batch_s<float, true>(t, a);
  }
  if (t.ts > 1) {
    if (prec == LBM_PREC_F64) return launch_batch_pipe_s<double>(t, a);
    if (prec == LBM_PREC_F32DEV) return launch_batch_pipe_s<float>(t, a);
    if (prec == LBM_PREC_F32DEV_F64) return launch_batch_pipe_s<f32s_f64a>(t, a);
    return launch_batch_pipe_s<__half>(t, a);
  }
  if (prec == LBM_PREC_F64) return launch_batch_s<double>(t, a);
  if (prec == LBM_PREC_F32DEV) return launch_batch_s<float>(t, a);
  if (prec == LBM_PREC_F32DEV_F64) return launch_batch_s<f32s_f64a>(t, a);
  return launch_batch_s<__half>(t, a);
}

// Rows per block (two more are pulled for psi): 2048 blocks or more, so that every CU
// has 8, but 2 to 16 rows.  Measured: 700 x 300 FP64 7.0 us with 4 rows, 10.3 with 8, 31
// with 32; 2048 x 2048 FP64 101, 98, 101, 120 us with 8, 16, 32, 64; FP16 39, 43, 53 with
// 8, 16, 32; 4096 x 4096 FP64 417, 404, 408 with 8, 16, 32.
template <typename S>
hipError_t launch_fields_s(const void* src, const RunDev& d, double* rho, double* vx, double* vy, double* p,
                           hipStream_t st) {
  const int threads = d.nx <= 62 ? 64 : d.nx <= 126 ? 128 : 256;
  const int64_t nstrips = (d.nx + threads - 3) / (threads - 2);
  const int64_t L = std::min<int64_t>(d.ny, std::min<int64_t>(16, std::max<int64_t>(2, nstrips * d.ny / 2048)));
  const int64_t grid = nstrips * ((d.ny + L - 1) / L);
  hipLaunchKernelGGL(k_fields<S>, dim3((unsigned)grid), dim3(threads), 0, st,
                     static_cast<const typename Store<S>::E*>(src), d, (int)L, (int)nstrips, rho, vx, vy, p);
  return hipGetLastError();
}

hipError_t launch_moments(int prec, const void* src, const RunDev& d, double* rho, double* vx,
                          double* vy, double* p, hipStream_t st) {
  if (prec == LBM_PREC_F64) return launch_fields_s<double>(src, d, rho, vx, vy, p, st);
  if (prec == LBM_PREC_F32DEV) return launch_fields_s<float>(src, d, rho, vx, vy, p, st);
  if (prec == LBM_PREC_F32DEV_F64) return launch_fields_s<f32s_f64a>(src, d, rho, vx, vy, p, st);
  return launch_fields_s<__half>(src, d, rho, vx, vy, p, st);
}

// Mass partials of kMassBlocks work-groups into part_i/part_d, then the final
// sums into out[0..2] and *flag (nullable) into out[3] (see k_mass_final).
hipError_t launch_mass(int prec, const void* src, const RunDev& d, __int128* pi, double* pd,
                       const unsigned long long* flag, unsigned long long* out, hipStream_t st) {
  if (prec == LBM_PREC_F64)
    hipLaunchKernelGGL(k_mass<double>, dim3(kMassBlocks), dim3(256), 0, st, (const double*)src, d, pi, pd);
  else if (prec == LBM_PREC_F32DEV)
    hipLaunchKernelGGL(k_mass<float>, dim3(kMassBlocks), dim3(256), 0, st, (const float*)src, d, pi, pd);
  else if (prec == LBM_PREC_F32DEV_F64)
    hipLaunchKernelGGL(k_mass<f32s_f64a>, dim3(kMassBlocks), dim3(256), 0, st, (const float*)src, d, pi, pd);
  else
    hipLaunchKernelGGL(k_mass<__half>, dim3(kMassBlocks), dim3(256), 0, st, (const __half*)src, d, pi, pd);
  hipLaunchKernelGGL(k_mass_final, dim3(1), dim3(256), 0, st, (const __int128*)pi, (const double*)pd,
                     kMassBlocks, flag, out);
  return hipGetLastError();
}

// Bytes of mass scratch: 128-bit and FP64 partials per work-group, then the
// four result words.
constexpr size_t kMassScratch = kMassBlocks * (sizeof(__int128) + sizeof(double)) + 4 * sizeof(unsigned long long);

}  // namespace
}  // namespace lbm

// Device scratch of lbm_mass_noalloc (the mass partials and result words,
// kMassScratch = 24,608 bytes), one copy per GPU, held until the process ends.
// Host code never uses this name as an address: it uses the per-device
// pointer hipGetSymbolAddress returned for it.
static __device__ __align__(256) unsigned char scratch[lbm::kMassScratch];

namespace lbm {
namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices];  // device address of `scratch` per device (null until set up)

// The current device's address of `scratch`, looked up on the first call on
// that device (with it current) and kept.
hipError_t scratch_of_current_device(char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch[dev] = p;
  }
  *out = static_cast<char*>(g_scratch[dev]);
  return hipSuccess;
}

hipError_t launch_batch_coex(int prec, const void* pool, const RunDev* runs, int nruns,
                             const unsigned long long* flags, double* out, hipStream_t st) {
  const dim3 g(nruns), b(256);
  if (prec == LBM_PREC_F64)
    hipLaunchKernelGGL(k_batch_coex<double>, g, b, 0, st, (const double*)pool, runs, flags, out);
  else if (prec == LBM_PREC_F32DEV)
    hipLaunchKernelGGL(k_batch_coex<float>, g, b, 0, st, (const float*)pool, runs, flags, out);
  else if (prec == LBM_PREC_F32DEV_F64)
    hipLaunchKernelGGL(k_batch_coex<f32s_f64a>, g, b, 0, st, (const float*)pool, runs, flags, out);
  else
    hipLaunchKernelGGL(k_batch_coex<__half>, g, b, 0, st, (const __half*)pool, runs, flags, out);
  return hipGetLastError();
}

// ---- tile heuristics and tuning cache -----------------------------------------

Tile default_tile(int nx, int ny) {
  Tile t{nx >= 1024 ? 4 : nx >= 256 ? 2 : 1, 0, 2};
  const int SW = 64 * t.nw;
  const int64_t rows = (int64_t)((nx + SW - 1) / SW) * ny;
  if (rows < 8 * 1024) {  // small lattices: short chunks give more blocks
    int l = 64;
    while (l > 4 && ((nx + SW - 1) / SW) * ((ny + l - 1) / l) < 1024) l /= 2;
    t.L = std::min(l, std::max(1, ny));
  }
  return t;
}

// A tile and what runs the steps that it leaves over: rem[r - 1] is the launch with r steps
// to go, r < t.ts (of r steps or fewer).
struct Plan {
  Tile t;
  Tile rem[3];
  const Tile& next(int64_t left) const { return left >= t.ts ? t : rem[left - 1]; }
};

// Tuned plans by size and kind, for the life of the process.  Lattices and batches have a
// map each: their keys are of one type, and a tile of the one is not always one of the other.
using TuneKey = std::tuple<int, int, int, int>;
std::mutex g_tune_mu;
std::map<TuneKey, Plan> g_tune, g_batch_tune;

}  // namespace
}  // namespace lbm

using namespace lbm;

struct lbm_ctx {
  lbm_params p;
  EosConst k;
  RunDev d;
  int esize;
  size_t pop_bytes, raw_bytes;
  char* ws;
  size_t ws_bytes;
  void* buf[2];
  int cur;
  double* aux;  // 4 planes of nx*ny doubles: rho, vx, vy, p
  __int128* part_i;   // mass scratch: partials and the result words
  double* part_d;
  unsigned long long* mass_out;
  unsigned long long* flag;
  unsigned long long* ctr;
  hipStream_t st;
  int64_t step;
  Plan plan;
  int graph_k;
  hipGraphExec_t gexec[2];
  Plan gplan;
  int64_t captures;  // graphs captured so far
};

namespace {

size_t raw_bytes_of(const lbm_params& p) {
  const int es = esize_of(p.precision);
  return (size_t)elems_of(p.nx, p.ny) * es;
}

size_t ctx_layout(const lbm_params& p, size_t* pop, size_t* aux, size_t* parts, size_t* misc) {
  *pop = align_up(raw_bytes_of(p));
  *aux = align_up(4 * (size_t)p.nx * p.ny * sizeof(double));
  *parts = align_up(kMassScratch);
  *misc = align_up(2 * sizeof(unsigned long long));
  return 2 * *pop + *aux + *parts + *misc;
}

bool same_tile(const Tile& a, const Tile& b) {
  return a.nw == b.nw && a.L == b.L && a.pf == b.pf && a.ts == b.ts;
}

// A launch shape.  Multi-step tiles: strip class nw 4 (8 is the same) or 2 (narrow
// strips: batches, and single lattices at four steps), or patches (nw 1, no rows; single
// lattices); three steps only for single lattices.  More than two steps and patches: depth 1.
bool valid_tile(int nw, int L, int pf, int maxnw, int ts = 1, bool batch = false) {
  const bool patch = nw == 1 && L == 0 && pf == 1 && !batch;
  if (ts > 1 && nw != 4 && nw != 8 && !(nw == 2 && (batch || ts == 4)) && !patch) return false;
  if (ts == 3 && batch) return false;
  if (ts > 2 && pf != 1) return false;
  return (nw == 1 || nw == 2 || nw == 4 || nw == 8 || nw == 16) && nw <= maxnw && L >= 0 &&
         L <= LMAX && (pf == 1 || pf == 2) && ts >= 1 && ts <= 4;
}

// Tile t with ts steps per launch (a remainder; a patch's single step takes one-row
// chunks, which give a small lattice the most blocks).
Tile with_steps(Tile t, int ts) {
  if (t.nw == 1 && t.ts > 1 && ts == 1) t.L = 1;
  t.ts = ts;
  return t;
}

// The plan of a tile that was not tuned: its own shape with fewer steps (three only where
// that kernel exists: single lattices' patches and FP64 arithmetic).
Plan plan_of(int prec, const Tile& t, bool batch = false) {
  Plan p{t, {t, t, t}};
  const bool three = !batch && (t.nw == 1 || has_step3(prec));
  for (int r = 1; r < t.ts; ++r) p.rem[r - 1] = with_steps(t, r == 3 && !three ? 2 : r);
  return p;
}

bool same_plan(const Plan& a, const Plan& b) {
  bool same = same_tile(a.t, b.t);
  for (int r = 1; same && r < a.t.ts; ++r) same = same_tile(a.rem[r - 1], b.rem[r - 1]);
  return same;
}

// The next launch of a lattice with `left` steps to go.  Single steps take the place of
// several where rows have 2^32 bytes and more (the pipe addresses a row with 32-bit byte
// offsets) and of patches that are too many for one launch.
Tile next_launch(const lbm_ctx* c, int64_t left) {
  const Tile& t = c->plan.next(left);
  if (t.ts == 1) return t;
  const bool fits = t.nw == 1 ? layout::launchable(layout::patches(c->p.nx, c->p.ny, t.ts), layout::patch_threads(t.ts))
                              : (int64_t)c->p.nx * c->esize < (1ll << 32);
  return fits ? t : with_steps(t, 1);
}

// Launches that k steps take.
int launches_of(const lbm_ctx* c, int k) {
  int n = 0;
  for (; k > 0; ++n) k -= next_launch(c, k).ts;
  return n;
}

void drop_graphs(lbm_ctx* c) {
  for (int i = 0; i < 2; ++i)
    if (c->gexec[i]) {
      (void)hipGraphExecDestroy(c->gexec[i]);
      c->gexec[i] = nullptr;
    }
}

int upload_state(lbm_ctx* c, const std::vector<char>& raw, int64_t step) {
  HIPCHK(hipMemcpyAsync(c->buf[0], raw.data(), raw.size(), hipMemcpyHostToDevice, c->st));
  c->cur = 0;
  c->step = step;
  hipLaunchKernelGGL(k_counter_set, dim3(1), dim3(1), 0, c->st, c->flag, kNoDiv);
  hipLaunchKernelGGL(k_counter_set, dim3(1), dim3(1), 0, c->st, c->ctr, (unsigned long long)step);
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(c->st));
  return LBM_OK;
}

int capture_graph(lbm_ctx* c, int parity) {
  hipGraph_t g;
  HIPCHK(hipStreamBeginCapture(c->st, hipStreamCaptureModeThreadLocal));
  hipError_t e = hipSuccess;
  for (int s = parity, done = 0; done < c->graph_k && e == hipSuccess; s ^= 1) {
    const Tile t = next_launch(c, c->graph_k - done);
    e = launch_step(c->p.precision, t, c->buf[s], c->buf[s ^ 1], c->d, c->ctr, (unsigned long long)done,
                    c->flag, c->st);
    done += t.ts;
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_counter_add, dim3(1), dim3(1), 0, c->st, c->ctr,
                       (unsigned long long)c->graph_k);
    e = hipGetLastError();
  }
  hipError_t e2 = hipStreamEndCapture(c->st, &g);
  if (e != hipSuccess || e2 != hipSuccess) return LBM_EHIP;
  e = hipGraphInstantiate(&c->gexec[parity], g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e == hipSuccess) e = hipGraphUpload(c->gexec[parity], c->st);
  if (e != hipSuccess) {
    if (c->gexec[parity]) (void)hipGraphExecDestroy(c->gexec[parity]);
    c->gexec[parity] = nullptr;
    return LBM_EHIP;
  }
  c->gplan = c->plan;
  ++c->captures;
  return LBM_OK;
}

// Capture (or re-capture after a tile change) the graphs of both buffer
// parities now, so that no later lbm_step call pays for a capture.
int prepare_graphs(lbm_ctx* c) {
  if (c->graph_k <= 0) return LBM_OK;
  if (!same_plan(c->gplan, c->plan)) drop_graphs(c);
  for (int parity = 0; parity < 2; ++parity)
    if (!c->gexec[parity]) {
      int st = capture_graph(c, parity);
      if (st != LBM_OK) return st;
    }
  HIPCHK(hipStreamSynchronize(c->st));
  return LBM_OK;
}

// Time `reps` launches of one candidate tile (reads the current buffer, writes
// the other, so the state does not advance).  Returns ms or a negative value.
template <class Launch>
float time_launches(hipStream_t st, Launch&& launch, int reps) {
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return -1.f;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return -1.f;
  }
  hipError_t e = hipSuccess;
  for (int r = 0; r < 2 && e == hipSuccess; ++r) e = launch();
  if (e == hipSuccess) e = hipEventRecord(e0, st);
  for (int r = 0; r < reps && e == hipSuccess; ++r) e = launch();
  if (e == hipSuccess) e = hipEventRecord(e1, st);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float ms = -1.f;
  if (e == hipSuccess && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) ms = -1.f;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return e == hipSuccess ? ms : -1.f;
}

// Pick the fastest tile per lattice step (tuning::pick_best), and for fewer steps than it
// takes the launches whose times add up to the least.  time_one(t) returns ms per lattice
// step, negative on a HIP error, +inf to skip the tile.  Returns LBM_OK (plan unchanged if
// every tile was skipped) or LBM_EHIP.
template <class TimeOne>
int pick_plan(int prec, bool batch, const std::vector<Tile>& cand, TimeOne&& time_one, Plan& plan) {
  const int n = (int)cand.size();
  std::vector<float> least(n, 1e30f);
  const int k = tuning::pick_best(n, [&](int i) {
    const float ms = time_one(cand[i]);
    if (ms >= 0) least[i] = std::min(least[i], ms);
    return ms;
  });
  if (k == -2) return LBM_EHIP;
  if (k < 0) return LBM_OK;
  plan = plan_of(prec, cand[k], batch);
  float cost[4] = {};  // of r steps
  for (int r = 1; r < plan.t.ts; ++r) {
    cost[r] = 1e30f;
    for (int i = 0; i < n; ++i) {
      const int ts = cand[i].ts;
      if (ts > r || least[i] >= 1e30f || least[i] * ts + cost[r - ts] >= cost[r]) continue;
      cost[r] = least[i] * ts + cost[r - ts];
      plan.rem[r - 1] = cand[i];
    }
  }
  return LBM_OK;
}

}  // namespace

extern "C" {

const char* lbm_strerror(int s) {
  switch (s) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument";
    case LBM_EPSI: return "density outside the equation-of-state range (2(p - rho/3)/G <= 0)";
    case LBM_EDIVERGED: return "the run diverged";
    case LBM_EHIP: return "HIP runtime error";
    case LBM_ENOSPACE: return "workspace too small";
    case LBM_ENOTSUP: return "not supported";
    default: return "unknown error";
  }
}

int lbm_workspace_bytes(const lbm_params* p, size_t* bytes) {
  if (!p || !bytes) return LBM_EINVAL;
  int st = validate(*p);
  if (st != LBM_OK) return st;
  size_t a, b, c2, d2;
  *bytes = ctx_layout(*p, &a, &b, &c2, &d2);
  return LBM_OK;
}

int lbm_init(const lbm_params* p, const double* rho0, const double* ux0, const double* uy0,
             void* ws, size_t ws_bytes, void* stream, lbm_ctx** out) {
  if (!p || !rho0 || !ws || !out) return LBM_EINVAL;
  *out = nullptr;
  int st = validate(*p);
  if (st != LBM_OK) return st;
  if (reinterpret_cast<uintptr_t>(ws) % kAlign) return LBM_EINVAL;
  size_t pop, aux, parts, misc;
  const size_t need = ctx_layout(*p, &pop, &aux, &parts, &misc);
  if (ws_bytes < need) return LBM_ENOSPACE;
  EosConst k;
  st = eos_constants(*p, &k);
  if (st != LBM_OK) return st;
  const size_t n = (size_t)p->nx * p->ny;
  double mean = 0.0;
  for (size_t i = 0; i < n; ++i) {
    if (!(rho0[i] > 0) || !(host_psi2(k, rho0[i]) > 0)) return LBM_EPSI;
    mean += rho0[i];
  }
  mean /= (double)n;
  double rref = 0.0;
  if (p->precision != LBM_PREC_F64) rref = std::isnan(p->rho_ref) ? mean : p->rho_ref;
  std::vector<double> f(9 * n);
  for (size_t i = 0; i < n; ++i) {
    double fe[9];
    host_feq(rho0[i], ux0 ? ux0[i] : 0.0, uy0 ? uy0[i] : 0.0, fe);
    for (int a = 0; a < 9; ++a) f[a * n + i] = fe[a];
  }
  lbm_ctx* c = new lbm_ctx{};
  c->p = *p;
  c->p.rho_ref = rref;
  c->k = k;
  c->d = make_rundev(*p, k, rref, 0, 0);
  c->esize = esize_of(p->precision);
  c->pop_bytes = pop;
  c->raw_bytes = raw_bytes_of(*p);
  c->ws = static_cast<char*>(ws);
  c->ws_bytes = ws_bytes;
  c->buf[0] = c->ws;
  c->buf[1] = c->ws + pop;
  c->aux = reinterpret_cast<double*>(c->ws + 2 * pop);
  c->part_i = reinterpret_cast<__int128*>(c->ws + 2 * pop + aux);
  c->part_d = reinterpret_cast<double*>(c->part_i + kMassBlocks);
  c->mass_out = reinterpret_cast<unsigned long long*>(c->part_d + kMassBlocks);
  c->flag = reinterpret_cast<unsigned long long*>(c->ws + 2 * pop + aux + parts);
  c->ctr = c->flag + 1;
  c->st = static_cast<hipStream_t>(stream);
  c->plan = plan_of(p->precision, default_tile(p->nx, p->ny));
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune.find({p->nx, p->ny, p->precision, 0});
    if (it != g_tune.end()) c->plan = it->second;
  }
  // the second buffer is written only at lattice nodes: clear its row padding once
  // so that checkpoints of either buffer are deterministic
  if (hipMemsetAsync(c->buf[1], 0, c->raw_bytes, c->st) != hipSuccess) {
    delete c;
    return LBM_EHIP;
  }
  std::vector<char> raw;
  encode_any(p->precision, c->p, rref, f.data(), raw);
  st = upload_state(c, raw, 0);
  if (st != LBM_OK) {
    delete c;
    return st;
  }
  *out = c;
  return LBM_OK;
}

int lbm_step(lbm_ctx* c, int64_t n) {
  if (!c || n < 0) return LBM_EINVAL;
  int64_t done = 0;
  if (c->graph_k > 0 && n >= c->graph_k) {
    if (!same_plan(c->gplan, c->plan)) drop_graphs(c);
    hipLaunchKernelGGL(k_counter_set, dim3(1), dim3(1), 0, c->st, c->ctr, (unsigned long long)c->step);
    HIPCHK(hipGetLastError());
    while (n - done >= c->graph_k) {
      if (!c->gexec[c->cur]) {
        int st = capture_graph(c, c->cur);
        if (st != LBM_OK) return st;
      }
      HIPCHK(hipGraphLaunch(c->gexec[c->cur], c->st));
      done += c->graph_k;
      c->step += c->graph_k;
      c->cur ^= launches_of(c, c->graph_k) & 1;  // a buffer swap each
    }
  }
  while (done < n) {
    const int s = c->cur;
    const Tile t = next_launch(c, n - done);
    HIPCHK(launch_step(c->p.precision, t, c->buf[s], c->buf[s ^ 1], c->d, nullptr,
                       (unsigned long long)c->step, c->flag, c->st));
    c->cur ^= 1;
    c->step += t.ts;
    done += t.ts;
  }
  return LBM_OK;
}

int lbm_status(lbm_ctx* c, int64_t* step, int64_t* diverged_at) {
  if (!c) return LBM_EINVAL;
  unsigned long long f = 0;
  HIPCHK(hipMemcpyAsync(&f, c->flag, sizeof f, hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  if (step) *step = c->step;
  if (diverged_at) *diverged_at = f == kNoDiv ? -1 : (int64_t)f;
  return f == kNoDiv ? LBM_OK : LBM_EDIVERGED;
}

int lbm_moments_device(lbm_ctx* c, double* rho, double* vx, double* vy, double* p) {
  if (!c || !rho || !vx || !vy || !p) return LBM_EINVAL;
  HIPCHK(launch_moments(c->p.precision, c->buf[c->cur], c->d, rho, vx, vy, p, c->st));
  return LBM_OK;
}

int lbm_moments(lbm_ctx* c, double* rho, double* vx, double* vy, double* p) {
  if (!c) return LBM_EINVAL;
  const size_t n = (size_t)c->p.nx * c->p.ny;
  double* a = c->aux;
  int st = lbm_moments_device(c, a, a + n, a + 2 * n, a + 3 * n);
  if (st != LBM_OK) return st;
  double* outs[4] = {rho, vx, vy, p};
  for (int i = 0; i < 4; ++i)
    if (outs[i]) HIPCHK(hipMemcpyAsync(outs[i], a + i * n, n * sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  return lbm_status(c, nullptr, nullptr);
}

int lbm_flat_profile(lbm_ctx* c, double* rho_bar, double* p_n) {
  if (!c || !rho_bar) return LBM_EINVAL;
  if (p_n && (c->p.scheme != LBM_SCHEME_IMPROVED || c->d.mrt)) return LBM_ENOTSUP;
  const size_t n = (size_t)c->p.nx * c->p.ny;
  double* a = c->aux;
  // rho plane at a; the column means and the pressure reuse the velocity plane
  double* rb = a + n;
  double* pn = rb + c->p.nx;
  HIPCHK(launch_moments(c->p.precision, c->buf[c->cur], c->d, a, a + n, a + 2 * n, a + 3 * n,
                        c->st));
  const dim3 blk(256), grd((c->p.nx + 255) / 256);
  hipLaunchKernelGGL(k_colmean, grd, blk, 0, c->st, (const double*)a, c->p.nx, c->p.ny, rb);
  if (p_n)
    hipLaunchKernelGGL(k_normal_pressure, grd, blk, 0, c->st, (const double*)rb, c->d, c->p.sigma, pn);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(rho_bar, rb, c->p.nx * sizeof(double), hipMemcpyDeviceToHost, c->st));
  if (p_n) HIPCHK(hipMemcpyAsync(p_n, pn, c->p.nx * sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  return lbm_status(c, nullptr, nullptr);
}

// The first three result words of the mass kernels into the caller's outputs.
static void mass_words(const unsigned long long* w, int64_t* fixed, double* mass) {
  if (fixed) {
    fixed[0] = (int64_t)w[0];
    fixed[1] = (int64_t)w[1];
  }
  if (mass) std::memcpy(mass, &w[2], sizeof(double));
}

int lbm_surface_tension(lbm_ctx* c, double* gamma) {
  if (!c || !gamma) return LBM_EINVAL;
  if (c->p.scheme != LBM_SCHEME_IMPROVED) return LBM_ENOTSUP;
  const size_t n = (size_t)c->p.nx * c->p.ny;
  double* a = c->aux;
  double* rb = a + n;  // column means and the result reuse the velocity plane
  double* g = rb + c->p.nx;
  HIPCHK(launch_moments(c->p.precision, c->buf[c->cur], c->d, a, a + n, a + 2 * n, a + 3 * n,
                        c->st));
  hipLaunchKernelGGL(k_colmean, dim3((c->p.nx + 255) / 256), dim3(256), 0, c->st, (const double*)a,
                     c->p.nx, c->p.ny, rb);
  hipLaunchKernelGGL(k_surface_tension, dim3(1), dim3(256), 0, c->st, (const double*)rb, c->d,
                     c->p.sigma, g);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(gamma, g, sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  return lbm_status(c, nullptr, nullptr);
}

int lbm_mass(lbm_ctx* c, int64_t* fixed, double* mass) {
  if (!c) return LBM_EINVAL;
  HIPCHK(launch_mass(c->p.precision, c->buf[c->cur], c->d, c->part_i, c->part_d, c->flag, c->mass_out, c->st));
  unsigned long long w[4];
  HIPCHK(hipMemcpyAsync(w, c->mass_out, sizeof w, hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  mass_words(w, fixed, mass);
  return w[3] == kNoDiv ? LBM_OK : LBM_EDIVERGED;
}

int lbm_mass_noalloc(const void* dev_populations, int32_t nx, int32_t ny, int32_t precision,
                     double rho_ref, void* hip_stream, int64_t* fixed, double* mass) {
  if (!dev_populations || nx < 3 || ny < 3) return LBM_EINVAL;
  if (precision < LBM_PREC_F64 || precision > LBM_PREC_F32DEV_F64 || !std::isfinite(rho_ref))
    return LBM_EINVAL;
  if ((int64_t)nx * ny > LBM_NOALLOC_MAX_NODES) return LBM_ENOSPACE;
  char* base = nullptr;
  HIPCHK(scratch_of_current_device(&base));
  RunDev d{};
  d.nx = nx;
  d.ny = ny;
  d.pitch = pitch_of(nx);
  d.plane = plane_of(nx);
  d.rs = rs_of(nx);
  d.elems = elems_of(nx, ny);
  d.rho_ref = precision == LBM_PREC_F64 ? 0.0 : rho_ref;
  __int128* pi = reinterpret_cast<__int128*>(base);
  double* pd = reinterpret_cast<double*>(pi + kMassBlocks);
  unsigned long long* out = reinterpret_cast<unsigned long long*>(pd + kMassBlocks);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  HIPCHK(launch_mass(precision, dev_populations, d, pi, pd, nullptr, out, st));
  unsigned long long w[3];
  HIPCHK(hipMemcpyAsync(w, out, sizeof w, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  mass_words(w, fixed, mass);
  return LBM_OK;
}

int lbm_get_populations(lbm_ctx* c, double* f, int64_t* step) {
  if (!c || !f) return LBM_EINVAL;
  std::vector<char> raw(c->raw_bytes);
  HIPCHK(hipMemcpyAsync(raw.data(), c->buf[c->cur], raw.size(), hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  decode_any(c->p.precision, c->p, c->p.rho_ref, raw.data(), f);
  if (step) *step = c->step;
  return lbm_status(c, nullptr, nullptr);
}

int lbm_set_populations(lbm_ctx* c, const double* f, int64_t step) {
  if (!c || !f || step < 0) return LBM_EINVAL;
  std::vector<char> raw;
  encode_any(c->p.precision, c->p, c->p.rho_ref, f, raw);
  return upload_state(c, raw, step);
}

// Checkpoint: a header {magic, version, step, precision, nx, ny, rho_ref, raw
// bytes} followed by the raw storage of the current buffer.
struct CkptHeader {
  uint64_t magic, version;
  int64_t step;
  int32_t precision, nx, ny, pad;
  double rho_ref;
  uint64_t raw_bytes;
};
static_assert(sizeof(CkptHeader) == 56, "header layout");
constexpr uint64_t kCkptMagic = 0x4C424D434B505431ull;

int lbm_state_bytes(lbm_ctx* c, size_t* bytes) {
  if (!c || !bytes) return LBM_EINVAL;
  *bytes = sizeof(CkptHeader) + c->raw_bytes;
  return LBM_OK;
}

int lbm_save_state(lbm_ctx* c, void* host, size_t bytes) {
  if (!c || !host || bytes < sizeof(CkptHeader) + c->raw_bytes) return LBM_EINVAL;
  CkptHeader h{kCkptMagic, 2, c->step, c->p.precision, c->p.nx, c->p.ny, 0, c->p.rho_ref, c->raw_bytes};
  std::memcpy(host, &h, sizeof h);
  HIPCHK(hipMemcpyAsync(static_cast<char*>(host) + sizeof h, c->buf[c->cur], c->raw_bytes,
                        hipMemcpyDeviceToHost, c->st));
  HIPCHK(hipStreamSynchronize(c->st));
  return LBM_OK;
}

int lbm_load_state(lbm_ctx* c, const void* host, size_t bytes) {
  if (!c || !host || bytes < sizeof(CkptHeader)) return LBM_EINVAL;
  CkptHeader h;
  std::memcpy(&h, host, sizeof h);
  if (h.magic != kCkptMagic || h.version != 2 || h.precision != c->p.precision || h.nx != c->p.nx ||
      h.ny != c->p.ny || h.raw_bytes != c->raw_bytes || bytes < sizeof h + c->raw_bytes ||
      !(h.rho_ref == c->p.rho_ref) || h.step < 0)
    return LBM_EINVAL;
  std::vector<char> raw(static_cast<const char*>(host) + sizeof h,
                        static_cast<const char*>(host) + sizeof h + c->raw_bytes);
  return upload_state(c, raw, h.step);
}

int lbm_set_tile(lbm_ctx* c, int32_t nw, int32_t L, int32_t depth, int32_t steps) {
  if (!c || !valid_tile(nw, L, depth, 16, steps)) return LBM_EINVAL;
  if (steps == 3 && nw != 1 && !has_step3(c->p.precision)) return LBM_ENOTSUP;
  if (steps == 3 && nw != 1 && (c->p.nx < 5 || c->p.ny < 5)) return LBM_EINVAL;
  c->plan = plan_of(c->p.precision, Tile{nw, L, depth, steps});
  return prepare_graphs(c);
}

int lbm_get_tile(lbm_ctx* c, int32_t* nw, int32_t* L, int32_t* depth, int32_t* steps) {
  if (!c) return LBM_EINVAL;
  if (nw) *nw = c->plan.t.nw;
  if (L) *L = c->plan.t.L;
  if (depth) *depth = c->plan.t.pf;
  if (steps) *steps = c->plan.t.ts;
  return LBM_OK;
}

int lbm_tune(lbm_ctx* c, int32_t* nw_out, int32_t* L_out, int32_t* depth_out, int32_t* steps_out) {
  if (!c) return LBM_EINVAL;
  Plan best = c->plan;
  const int s = c->cur;
  const int64_t nodes = (int64_t)c->p.nx * c->p.ny;
  const int reps = nodes >= (1 << 22) ? 3 : 10;
  std::vector<Tile> cand;
  // Tuning is most of the time it takes to set a lattice up, so of each family only the
  // likeliest are timed.  Patches win below 2^16 nodes by 1.8 times and more and lose
  // above 2^18.  Single steps win on narrow lattices only, but are what a program takes that
  // reads its lattice after every step.  Of all their tiles the fastest had chunks of one or
  // two rows up to 2^18 nodes (depth 2: 64 x 32 4.0 us, depth 1 4.6), two to four up to 2^20,
  // with one wave on the smallest and on narrow lattices and up to 16 on others (1024 x 1024
  // FP16 13.7 us with 16, 13.9 with 4), and the balanced schedule from 2^21 on.
  // Strips twice as wide as the lattice and more are left out, and pipes that use less than a
  // quarter of their lanes.
  const bool tiny = nodes < (1 << 16), large = nodes >= (1 << 21);
  auto one = [&](int nw, int L, int pf) {
    if (nw == 1 || 32 * nw < c->p.nx) cand.push_back(Tile{nw, std::min(L, 2 * c->p.ny), pf, 1});
  };
  if (nodes <= (1 << 18))
    for (int ts : {2, 3, 4}) cand.push_back(Tile{1, 0, 1, ts});
  if (tiny) {
    for (int pf : {1, 2})
      for (int L : {1, 2}) one(1, L, pf);
  } else if (!large) {
    int rows = 1;
    while (2 * rows <= (nodes >> 18)) rows *= 2;
    for (int nw : {1, 2, 4, 8, 16})
      for (int L : {rows, 2 * rows}) one(nw, L, rows == 1 ? 2 : 1);
  } else {
    one(1, 0, 2);
    one(1, 64, 2);
    one(4, 8, 2);
    one(16, 0, 1);
  }
  if (!tiny) one(4, 0, 2);
  const bool narrow = c->p.nx >= 32, wide = c->p.nx > 114;  // 114: one narrow strip of four steps
  if ((int64_t)c->p.nx * c->esize < (1ll << 32))
    for (int L : {0, 16, 32, 64, 128})
      if (L <= 2 * c->p.ny && (!tiny || L == 16)) {
        if (wide) cand.push_back(Tile{4, L, 1, 4});
        if (narrow) cand.push_back(Tile{2, L, 1, 4});
        if (wide && (L == 0 || L == 32)) cand.push_back(Tile{4, L, 1, 2});
        if (wide && L == 0 && has_step3(c->p.precision) && c->p.ny >= 5) cand.push_back(Tile{4, 0, 1, 3});
      }
  const int pst = pick_plan(
      c->p.precision, false, cand,
      [&](const Tile& t) {
        const float ms = time_launches(
            c->st,
            [&] {
              return launch_step(c->p.precision, t, c->buf[s], c->buf[s ^ 1], c->d, nullptr,
                                 (unsigned long long)c->step, c->flag, c->st);
            },
            reps);
        return ms < 0 ? ms : ms / t.ts;  // time per lattice step
      },
      best);
  if (pst != LBM_OK) return pst;
  c->plan = best;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[{c->p.nx, c->p.ny, c->p.precision, c->d.mrt}] = best;
  }
  const int gst = prepare_graphs(c);
  if (gst != LBM_OK) return gst;
  if (nw_out) *nw_out = best.t.nw;
  if (L_out) *L_out = best.t.L;
  if (depth_out) *depth_out = best.t.pf;
  if (steps_out) *steps_out = best.t.ts;
  return LBM_OK;
}

int lbm_set_graph_steps(lbm_ctx* c, int32_t k) {
  if (!c || k < 0 || (k > 0 && (k < 2 || k % 2))) return LBM_EINVAL;
  if (k > 0 && c->st == nullptr) return LBM_EINVAL;  // the null stream cannot be captured
  drop_graphs(c);
  c->graph_k = k;
  return prepare_graphs(c);
}

int lbm_set_mrt(lbm_ctx* c, const double* rates) {
  if (!c) return LBM_EINVAL;
  if (!rates) {
    const int mrt = c->d.mrt;
    c->d = make_rundev(c->p, c->k, c->p.rho_ref, 0, 0);
    if (mrt) drop_graphs(c);
    return prepare_graphs(c);
  }
  if (c->p.scheme != LBM_SCHEME_IMPROVED) return LBM_ENOTSUP;
  if (c->p.precision != LBM_PREC_F64 && c->p.precision != LBM_PREC_F32DEV) return LBM_ENOTSUP;
  for (int i = 0; i < 3; ++i)
    if (!(rates[i] > 0.0 && rates[i] < 2.0)) return LBM_EINVAL;
  c->d = make_rundev(c->p, c->k, c->p.rho_ref, 0, 0);
  set_mrt(c->d, c->p, rates);
  drop_graphs(c);  // the captured launches carry the old constants
  return prepare_graphs(c);
}

int lbm_graph_captures(lbm_ctx* c, int64_t* n) {
  if (!c || !n) return LBM_EINVAL;
  *n = c->captures;
  return LBM_OK;
}

int lbm_debug_index_faults(uint64_t* count) {
  if (!count) return LBM_EINVAL;
#ifdef LBM_CHECK_INDEX
  unsigned long long v = 0, zero = 0;
  HIPCHK(hipDeviceSynchronize());
  HIPCHK(hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_index_faults), sizeof v));
  HIPCHK(hipMemcpyToSymbol(HIP_SYMBOL(g_index_faults), &zero, sizeof zero));
  *count = v;
  return LBM_OK;
#else
  *count = 0;
  return LBM_ENOTSUP;
#endif
}

int lbm_get_params(lbm_ctx* c, lbm_params* out) {
  if (!c || !out) return LBM_EINVAL;
  *out = c->p;
  return LBM_OK;
}

int lbm_device_buffers(lbm_ctx* c, void** b0, void** b1, int32_t* cur) {
  if (!c) return LBM_EINVAL;
  if (b0) *b0 = c->buf[0];
  if (b1) *b1 = c->buf[1];
  if (cur) *cur = c->cur;
  return LBM_OK;
}

int lbm_destroy(lbm_ctx* c) {
  if (!c) return LBM_EINVAL;
  (void)hipStreamSynchronize(c->st);
  drop_graphs(c);
  delete c;
  return LBM_OK;
}

}  // extern "C"

// ============================================================================
// Batch of independent lattices.
// ============================================================================

// The work list of one tile on the device: in item lists the blocks' first items (grid + 1
// entries), then all items.
struct WorkList {
  Item* d;
  int nitems, total;  // total: rows of the balanced schedule (0 for item lists)
  int grid;           // blocks the list was dealt to, or of the balanced schedule
};

struct lbm_batch {
  int nruns;
  int prec, esize;
  std::vector<lbm_params> p;
  std::vector<EosConst> k;
  std::vector<RunDev> d;  // host copy of the descriptor table
  std::vector<int64_t> nodes;
  char* ws;
  size_t pool_bytes;
  void* buf[2];
  int cur;
  RunDev* d_runs;
  WorkList list[3];  // of the tile, and of two and one step left over
  int items_cap;     // items of a list, without its blocks' first ones
  unsigned long long* flags;
  unsigned long long* ctr;
  double* aux;
  hipStream_t st;
  int64_t step;
  Plan plan;
  int graph_k;
  hipGraphExec_t gexec[2];
  Plan gplan;
  int64_t captures;  // graphs captured so far
  double* coex;      // 2 * nruns doubles: (rho_l, rho_g) per run
  int mrt;           // 1: every run's descriptor carries the MRT collision
};

namespace {

struct BatchLayout {
  size_t pool, runs, items, flags, aux, coex, total;
  int items_cap;
  size_t list_entries;  // of one of the three lists
};

int64_t run_elems(const lbm_params& q) { return layout::run_elems(q.nx, q.ny); }

BatchLayout batch_layout(int n, const lbm_params* p) {
  BatchLayout L{};
  size_t elems = 0, maxn = 0;
  int cap = 0;
  const size_t es = esize_of(p[0].precision);
  for (int i = 0; i < n; ++i) {
    elems += run_elems(p[i]);
    maxn = std::max(maxn, (size_t)p[i].nx * p[i].ny);
    cap += layout::max_items(p[i].nx, p[i].ny);
  }
  L.pool = align_up(elems * es);
  L.runs = align_up(n * sizeof(RunDev));
  L.items_cap = cap;
  L.list_entries = (size_t)cap + std::min(cap, kMaxBatchGrid) + 1;
  L.items = align_up(3 * L.list_entries * sizeof(Item));
  L.flags = align_up((n + 1) * sizeof(unsigned long long));
  L.aux = align_up(4 * maxn * sizeof(double));
  L.coex = align_up(2 * (size_t)n * sizeof(double));
  L.total = 2 * L.pool + L.runs + L.items + L.flags + L.aux + L.coex;
  return L;
}

// A launch of list l from buffer s into the other.
BatchArgs batch_args(const lbm_batch* b, const WorkList& l, int s, const unsigned long long* base,
                     unsigned long long local) {
  return BatchArgs{b->buf[s], b->buf[s ^ 1], b->d_runs, l.d, l.nitems, l.total,
                   l.grid,    base,          local,     b->flags, b->st, nullptr};
}

// Work list of a tile (layout::build_items, dealt to its kernel's grid or walked) into l and
// items; nothing on the device changes.
int make_list(const lbm_batch* b, const Tile& t, WorkList& l, std::vector<Item>& items) {
  std::vector<int> nx(b->nruns), ny(b->nruns);
  for (int r = 0; r < b->nruns; ++r) {
    nx[r] = b->p[r].nx;
    ny[r] = b->p[r].ny;
  }
  // multi-step strips: as wide as their kernel takes; those of FP64 lattices start on
  // 64-byte boundaries, as for a single lattice
  const bool f32 = b->prec == LBM_PREC_F32DEV || b->prec == LBM_PREC_F16DEV;  // FP32 arithmetic
  const int nw = t.ts == 1 ? t.nw : f32 ? pipe_nw<float>(t.nw) : pipe_nw<double>(t.nw);
  const int64_t rows = layout::build_items(b->nruns, nx.data(), ny.data(), nw, t.L, t.ts, items,
                                           b->prec == LBM_PREC_F64 ? StripAlign<double>::value : 1);
  if ((int)items.size() > b->items_cap) return LBM_ENOSPACE;
  if (rows >= INT32_MAX) return LBM_EINVAL;
  int resident = 1;
  BatchArgs q{};
  q.resident = &resident;
  HIPCHK(launch_batch(b->prec, b->mrt != 0, t, q));
  l.nitems = (int)items.size();
  l.total = t.L > 0 ? 0 : (int)rows;
  l.grid = batch_grid(resident, l.nitems, l.total);
  if (t.ts == 1 && t.L > 0 && t.L < layout::kWalkRows) layout::walk(items, l.grid);
  else if (t.L > 0) layout::deal(items, l.grid, t.ts > 1 ? pipe_fill(t.ts) : kStepFill);
  if (t.L > 0) layout::add_heads(items, l.grid);
  return LBM_OK;
}

// Enqueues the upload of a list; items must live until the stream has been waited for.
int upload_list(lbm_batch* b, const WorkList& l, const std::vector<Item>& items) {
  HIPCHK(hipMemcpyAsync(l.d, items.data(), items.size() * sizeof(Item), hipMemcpyHostToDevice, b->st));
  return LBM_OK;
}

// The lists of a plan: every launch has one dealt to the blocks that its own kernel keeps
// resident.  (With the tile's list and grid, one block per CU for four FP64 steps, single
// steps of a sweep of 256 runs took 111 us in FP64 and 53 in FP32; so 58 and 26.)
int batch_plan(lbm_batch* b, const Plan& p) {
  WorkList l[3] = {b->list[0], b->list[1], b->list[2]};
  std::vector<Item> items[3];
  int st = make_list(b, p.t, l[0], items[0]);
  for (int r = 1; r < p.t.ts && st == LBM_OK; ++r) {
    const Tile& t = p.rem[r - 1];
    if (items[3 - t.ts].empty()) st = make_list(b, t, l[3 - t.ts], items[3 - t.ts]);
  }
  for (int i = 0; i < 3 && st == LBM_OK; ++i)
    if (!items[i].empty()) st = upload_list(b, b->list[i] = l[i], items[i]);
  if (hipStreamSynchronize(b->st) != hipSuccess && st == LBM_OK) st = LBM_EHIP;
  if (st == LBM_OK) b->plan = p;
  return st;
}

// The next launch with `left` steps to go, and its list.
Tile batch_next(const lbm_batch* b, int64_t left, const WorkList** l) {
  const Tile& t = b->plan.next(left);
  *l = &b->list[left >= b->plan.t.ts ? 0 : 3 - t.ts];
  return t;
}

void batch_drop_graphs(lbm_batch* b) {
  for (int i = 0; i < 2; ++i)
    if (b->gexec[i]) {
      (void)hipGraphExecDestroy(b->gexec[i]);
      b->gexec[i] = nullptr;
    }
}

int batch_capture(lbm_batch* b, int parity) {
  hipGraph_t g;
  HIPCHK(hipStreamBeginCapture(b->st, hipStreamCaptureModeThreadLocal));
  hipError_t e = hipSuccess;
  for (int s = parity, done = 0; done < b->graph_k && e == hipSuccess; s ^= 1) {
    const WorkList* l;
    const Tile t = batch_next(b, b->graph_k - done, &l);
    e = launch_batch(b->prec, b->mrt != 0, t, batch_args(b, *l, s, b->ctr, (unsigned long long)done));
    done += t.ts;
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_counter_add, dim3(1), dim3(1), 0, b->st, b->ctr, (unsigned long long)b->graph_k);
    e = hipGetLastError();
  }
  hipError_t e2 = hipStreamEndCapture(b->st, &g);
  if (e != hipSuccess || e2 != hipSuccess) return LBM_EHIP;
  e = hipGraphInstantiate(&b->gexec[parity], g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e == hipSuccess) e = hipGraphUpload(b->gexec[parity], b->st);
  if (e != hipSuccess) {
    if (b->gexec[parity]) (void)hipGraphExecDestroy(b->gexec[parity]);
    b->gexec[parity] = nullptr;
    return LBM_EHIP;
  }
  b->gplan = b->plan;
  ++b->captures;
  return LBM_OK;
}

int batch_prepare_graphs(lbm_batch* b) {
  if (b->graph_k <= 0) return LBM_OK;
  if (!same_plan(b->gplan, b->plan)) batch_drop_graphs(b);
  for (int parity = 0; parity < 2; ++parity)
    if (!b->gexec[parity]) {
      int st = batch_capture(b, parity);
      if (st != LBM_OK) return st;
    }
  HIPCHK(hipStreamSynchronize(b->st));
  return LBM_OK;
}

TuneKey batch_key(const lbm_batch* b) {
  int64_t tot = 0;
  int maxnx = 0;
  for (int r = 0; r < b->nruns; ++r) {
    tot += b->nodes[r];
    maxnx = std::max(maxnx, b->p[r].nx);
  }
  return {(int)std::min<int64_t>(tot, INT32_MAX), maxnx, b->prec | (b->mrt << 8), b->nruns};
}

}  // namespace

extern "C" {

int lbm_batch_workspace_bytes(int32_t n, const lbm_params* p, size_t* bytes) {
  if (n < 1 || !p || !bytes) return LBM_EINVAL;
  for (int i = 0; i < n; ++i) {
    int st = validate(p[i]);
    if (st != LBM_OK) return st;
    if (p[i].precision != p[0].precision) return LBM_EINVAL;
  }
  *bytes = batch_layout(n, p).total;
  return LBM_OK;
}

int lbm_batch_init(int32_t n, const lbm_params* p, const double* const* rho0, void* ws,
                   size_t ws_bytes, void* stream, lbm_batch** out) {
  if (n < 1 || !p || !rho0 || !ws || !out) return LBM_EINVAL;
  *out = nullptr;
  size_t need;
  int st = lbm_batch_workspace_bytes(n, p, &need);
  if (st != LBM_OK) return st;
  if (ws_bytes < need) return LBM_ENOSPACE;
  if (reinterpret_cast<uintptr_t>(ws) % kAlign) return LBM_EINVAL;
  for (int r = 0; r < n; ++r)
    if (!rho0[r]) return LBM_EINVAL;
  const BatchLayout Lay = batch_layout(n, p);
  lbm_batch* b = new lbm_batch{};
  b->nruns = n;
  b->prec = p[0].precision;
  b->esize = esize_of(b->prec);
  b->p.assign(p, p + n);
  b->k.resize(n);
  b->ws = static_cast<char*>(ws);
  b->pool_bytes = Lay.pool;
  b->buf[0] = b->ws;
  b->buf[1] = b->ws + Lay.pool;
  b->d_runs = reinterpret_cast<RunDev*>(b->ws + 2 * Lay.pool);
  for (int i = 0; i < 3; ++i)
    b->list[i].d = reinterpret_cast<Item*>(b->ws + 2 * Lay.pool + Lay.runs) + i * Lay.list_entries;
  b->items_cap = Lay.items_cap;
  b->flags = reinterpret_cast<unsigned long long*>(b->ws + 2 * Lay.pool + Lay.runs + Lay.items);
  b->ctr = b->flags + n;
  b->aux = reinterpret_cast<double*>(b->ws + 2 * Lay.pool + Lay.runs + Lay.items + Lay.flags);
  b->coex = reinterpret_cast<double*>(b->ws + 2 * Lay.pool + Lay.runs + Lay.items + Lay.flags + Lay.aux);
  b->st = static_cast<hipStream_t>(stream);
  std::vector<char> pool(Lay.pool, 0);
  int64_t off = 0;
  for (int r = 0; r < n && st == LBM_OK; ++r) {
    const lbm_params& q = p[r];
    st = eos_constants(q, &b->k[r]);
    if (st != LBM_OK) break;
    const size_t nn = (size_t)q.nx * q.ny;
    double mean = 0;
    for (size_t i = 0; i < nn; ++i) {
      if (!(rho0[r][i] > 0) || !(host_psi2(b->k[r], rho0[r][i]) > 0)) st = LBM_EPSI;
      mean += rho0[r][i];
    }
    if (st != LBM_OK) break;
    mean /= (double)nn;
    const double rref = b->prec == LBM_PREC_F64 ? 0.0 : (std::isnan(q.rho_ref) ? mean : q.rho_ref);
    b->p[r].rho_ref = rref;
    b->d.push_back(make_rundev(q, b->k[r], rref, off, r));
    b->nodes.push_back((int64_t)nn);
    std::vector<double> f(9 * nn);
    for (size_t i = 0; i < nn; ++i) {
      double fe[9];
      host_feq(rho0[r][i], 0.0, 0.0, fe);
      for (int a = 0; a < 9; ++a) f[a * nn + i] = fe[a];
    }
    std::vector<char> raw;
    encode_any(b->prec, q, rref, f.data(), raw);
    std::memcpy(pool.data() + off * b->esize, raw.data(), raw.size());
    off += run_elems(q);
  }
  if (st != LBM_OK) {
    delete b;
    return st;
  }
  hipError_t e = hipMemcpyAsync(b->buf[0], pool.data(), pool.size(), hipMemcpyHostToDevice, b->st);
  if (e == hipSuccess) e = hipMemsetAsync(b->buf[1], 0, pool.size(), b->st);  // row padding
  if (e == hipSuccess)
    e = hipMemcpyAsync(b->d_runs, b->d.data(), n * sizeof(RunDev), hipMemcpyHostToDevice, b->st);
  std::vector<unsigned long long> fl(n + 1, kNoDiv);
  fl[n] = 0;  // step counter
  if (e == hipSuccess)
    e = hipMemcpyAsync(b->flags, fl.data(), fl.size() * sizeof(unsigned long long), hipMemcpyHostToDevice, b->st);
  if (e == hipSuccess) e = hipStreamSynchronize(b->st);
  if (e != hipSuccess) {
    delete b;
    return LBM_EHIP;
  }
  Plan plan = plan_of(b->prec, Tile{1, 16, 2}, true);
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_batch_tune.find(batch_key(b));
    if (it != g_batch_tune.end()) plan = it->second;
  }
  st = batch_plan(b, plan);
  if (st != LBM_OK) {
    delete b;
    return st;
  }
  *out = b;
  return LBM_OK;
}

int lbm_batch_step(lbm_batch* b, int64_t n) {
  if (!b || n < 0) return LBM_EINVAL;
  int64_t done = 0;
  if (b->graph_k > 0 && n >= b->graph_k) {
    if (!same_plan(b->gplan, b->plan)) batch_drop_graphs(b);
    hipLaunchKernelGGL(k_counter_set, dim3(1), dim3(1), 0, b->st, b->ctr, (unsigned long long)b->step);
    HIPCHK(hipGetLastError());
    while (n - done >= b->graph_k) {
      if (!b->gexec[b->cur]) {
        int st = batch_capture(b, b->cur);
        if (st != LBM_OK) return st;
      }
      HIPCHK(hipGraphLaunch(b->gexec[b->cur], b->st));
      done += b->graph_k;
      b->step += b->graph_k;
      for (int k = b->graph_k; k > 0; b->cur ^= 1) k -= b->plan.next(k).ts;  // a swap per launch
    }
  }
  while (done < n) {
    const int s = b->cur;
    const WorkList* l;
    const Tile t = batch_next(b, n - done, &l);
    HIPCHK(launch_batch(b->prec, b->mrt != 0, t, batch_args(b, *l, s, nullptr, (unsigned long long)b->step)));
    b->cur ^= 1;
    b->step += t.ts;
    done += t.ts;
  }
  return LBM_OK;
}

int lbm_batch_set_tile(lbm_batch* b, int32_t nw, int32_t L, int32_t depth, int32_t steps) {
  if (!b || !valid_tile(nw, L, depth, 8, steps, true) || (L > 0 && L < 4)) return LBM_EINVAL;
  batch_drop_graphs(b);
  const int st = batch_plan(b, plan_of(b->prec, Tile{nw, L, depth, steps}, true));
  return st != LBM_OK ? st : batch_prepare_graphs(b);
}

int lbm_batch_get_tile(lbm_batch* b, int32_t* nw, int32_t* L, int32_t* depth, int32_t* steps) {
  if (!b) return LBM_EINVAL;
  if (steps) *steps = b->plan.t.ts;
  if (nw) *nw = b->plan.t.nw;
  if (L) *L = b->plan.t.L;
  if (depth) *depth = b->plan.t.pf;
  return LBM_OK;
}

int lbm_batch_set_graph_steps(lbm_batch* b, int32_t k) {
  if (!b || k < 0 || (k > 0 && (k < 2 || k % 2))) return LBM_EINVAL;
  if (k > 0 && b->st == nullptr) return LBM_EINVAL;
  batch_drop_graphs(b);
  b->graph_k = k;
  return batch_prepare_graphs(b);
}

int lbm_batch_set_mrt(lbm_batch* b, const double* rates) {
  if (!b) return LBM_EINVAL;
  if (rates) {
    if (b->prec != LBM_PREC_F64 && b->prec != LBM_PREC_F32DEV) return LBM_ENOTSUP;
    for (int r = 0; r < b->nruns; ++r) {
      if (b->p[r].scheme != LBM_SCHEME_IMPROVED) return LBM_ENOTSUP;
      for (int i = 0; i < 3; ++i)
        if (!(rates[3 * r + i] > 0.0 && rates[3 * r + i] < 2.0)) return LBM_EINVAL;
    }
  }
  for (int r = 0; r < b->nruns; ++r) {
    RunDev& d = b->d[r];
    d.mrt = 0;
    if (rates) set_mrt(d, b->p[r], rates + 3 * r);
  }
  HIPCHK(hipMemcpyAsync(b->d_runs, b->d.data(), b->nruns * sizeof(RunDev), hipMemcpyHostToDevice, b->st));
  HIPCHK(hipStreamSynchronize(b->st));
  b->mrt = rates ? 1 : 0;
  batch_drop_graphs(b);  // the captured launches are of the other kernels
  const int st = batch_plan(b, b->plan);  // and so are the blocks that the lists were dealt to
  return st != LBM_OK ? st : batch_prepare_graphs(b);
}

int lbm_batch_graph_captures(lbm_batch* b, int64_t* n) {
  if (!b || !n) return LBM_EINVAL;
  *n = b->captures;
  return LBM_OK;
}

int lbm_batch_tune(lbm_batch* b, int32_t* nw_out, int32_t* L_out, int32_t* depth_out,
                   int32_t* steps_out) {
  if (!b) return LBM_EINVAL;
  Plan best = b->plan;
  const int s = b->cur;
  // as in lbm_tune, only the likeliest of each family
  std::vector<Tile> cand;
  for (int nw : {1, 2, 4})
    for (int L : {0, 4, 8, 16}) cand.push_back(Tile{nw, L, L == 4 ? 1 : 2, 1});
  for (int nw : {2, 4})
    for (int ts : {2, 4})
      for (int L : {0, 16, 32, 64}) cand.push_back(Tile{nw, L, 1, ts});  // 64: whole runs of a sweep
  int ist = LBM_OK;
  const int pst = pick_plan(
      b->prec, true, cand,
      [&](const Tile& t) {
        std::vector<Item> items;
        ist = make_list(b, t, b->list[0], items);
        if (ist == LBM_ENOSPACE) return 1e30f;  // too many items for the work list: skipped
        if (ist == LBM_OK) ist = upload_list(b, b->list[0], items);
        if (hipStreamSynchronize(b->st) != hipSuccess && ist == LBM_OK) ist = LBM_EHIP;
        if (ist != LBM_OK) return -1.f;
        const float ms = time_launches(
            b->st,
            [&] {
              return launch_batch(b->prec, b->mrt != 0, t,
                                  batch_args(b, b->list[0], s, nullptr, (unsigned long long)b->step));
            },
            5);
        return ms < 0 ? ms : ms / t.ts;  // time per lattice step
      },
      best);
  if (pst != LBM_OK) {
    (void)batch_plan(b, b->plan);  // the tile's own list again
    return ist != LBM_OK && ist != LBM_ENOSPACE ? ist : pst;
  }
  batch_drop_graphs(b);
  int st = batch_plan(b, best);
  if (st != LBM_OK) return st;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_batch_tune[batch_key(b)] = best;
  }
  st = batch_prepare_graphs(b);
  if (st != LBM_OK) return st;
  if (nw_out) *nw_out = best.t.nw;
  if (L_out) *L_out = best.t.L;
  if (depth_out) *depth_out = best.t.pf;
  if (steps_out) *steps_out = best.t.ts;
  return LBM_OK;
}

int lbm_batch_nodes(lbm_batch* b, int64_t* nodes) {
  if (!b || !nodes) return LBM_EINVAL;
  std::vector<unsigned long long> fl(b->nruns);
  HIPCHK(hipMemcpyAsync(fl.data(), b->flags, b->nruns * sizeof(unsigned long long), hipMemcpyDeviceToHost, b->st));
  HIPCHK(hipStreamSynchronize(b->st));
  int64_t t = 0;
  for (int r = 0; r < b->nruns; ++r)
    if (fl[r] == kNoDiv) t += b->nodes[r];
  *nodes = t;
  return LBM_OK;
}

// LBM_EDIVERGED when the run is frozen by divergence, else LBM_OK (synchronises).
static int batch_run_status(lbm_batch* b, int32_t run) {
  unsigned long long f = 0;
  HIPCHK(hipMemcpyAsync(&f, b->flags + run, sizeof f, hipMemcpyDeviceToHost, b->st));
  HIPCHK(hipStreamSynchronize(b->st));
  return f == kNoDiv ? LBM_OK : LBM_EDIVERGED;
}

int lbm_batch_moments(lbm_batch* b, int32_t run, double* rho, double* vx, double* vy, double* p) {
  if (!b || run < 0 || run >= b->nruns) return LBM_EINVAL;
  const RunDev& d = b->d[run];
  const size_t n = (size_t)d.nx * d.ny;
  double* a = b->aux;
  const char* src = static_cast<const char*>(b->buf[b->cur]) + d.off * b->esize;
  HIPCHK(launch_moments(b->prec, src, d, a, a + n, a + 2 * n, a + 3 * n, b->st));
  double* outs[4] = {rho, vx, vy, p};
  for (int i = 0; i < 4; ++i)
    if (outs[i]) HIPCHK(hipMemcpyAsync(outs[i], a + i * n, n * sizeof(double), hipMemcpyDeviceToHost, b->st));
  return batch_run_status(b, run);
}

int lbm_batch_get_populations(lbm_batch* b, int32_t run, double* f) {
  if (!b || run < 0 || run >= b->nruns || !f) return LBM_EINVAL;
  const RunDev& d = b->d[run];
  std::vector<char> raw(raw_bytes_of(b->p[run]));
  const char* src = static_cast<const char*>(b->buf[b->cur]) + d.off * b->esize;
  HIPCHK(hipMemcpyAsync(raw.data(), src, raw.size(), hipMemcpyDeviceToHost, b->st));
  const int st = batch_run_status(b, run);
  if (st != LBM_OK && st != LBM_EDIVERGED) return st;
  decode_any(b->prec, b->p[run], d.rho_ref, raw.data(), f);
  return st;
}

int lbm_batch_coexistence(lbm_batch* b, double* rho_l, double* rho_g, int32_t* status,
                          int64_t* diverged_at) {
  if (!b) return LBM_EINVAL;
  HIPCHK(launch_batch_coex(b->prec, b->buf[b->cur], b->d_runs, b->nruns, b->flags, b->coex, b->st));
  std::vector<unsigned long long> fl(b->nruns);
  std::vector<double> lg(2 * (size_t)b->nruns);
  HIPCHK(hipMemcpyAsync(fl.data(), b->flags, b->nruns * sizeof(unsigned long long), hipMemcpyDeviceToHost, b->st));
  HIPCHK(hipMemcpyAsync(lg.data(), b->coex, lg.size() * sizeof(double), hipMemcpyDeviceToHost, b->st));
  HIPCHK(hipStreamSynchronize(b->st));
  for (int r = 0; r < b->nruns; ++r) {
    const bool div = fl[r] != kNoDiv;
    if (status) status[r] = div ? LBM_EDIVERGED : LBM_OK;
    if (diverged_at) diverged_at[r] = div ? (int64_t)fl[r] : -1;
    if (rho_l) rho_l[r] = lg[2 * r];
    if (rho_g) rho_g[r] = lg[2 * r + 1];
  }
  return LBM_OK;
}

int lbm_batch_destroy(lbm_batch* b) {
  if (!b) return LBM_EINVAL;
  (void)hipStreamSynchronize(b->st);
  batch_drop_graphs(b);
  delete b;
  return LBM_OK;
}

}  // extern "C"
