// Device code of the fused pseudopotential D2Q9 step for gfx950.
//
// One work-group owns a strip of SW = 64*NW lattice columns (one column per
// thread) and a chunk of L rows, and marches up the chunk one row at a time:
//
//   * streaming is done on load (pull): f_a(x, y) = f*_a(x - e_a, y - e_a)
//     from the source buffer (paper Eq. 1);
//   * each loaded row gives rho and, in FP64, psi^2 = 2 (p_EOS - rho/3)/G
//     (Eqs. 8, 23); psi goes to a 4-row ring in LDS;
//   * the row below is then complete (psi at y-1, y, y+1), so its force
//     (Eq. 3), forcing scheme (Eqs. 9-11, 31) and BGK collision (Eqs. 1, 2)
//     are computed and its 9 populations stored, coalesced, to the
//     destination buffer at the same node.
//
// psi of the two halo columns x0-1 and x0+SW is computed once per chunk in a
// prologue; the halo rows y0-1 and y0+L are recomputed by the chunks on
// either side.  Populations are read once from HBM and written once (the
// neighbour strips' halo reads hit L2), so a step moves 2*9*sizeof(storage)
// bytes per node.  The paper gives no kernel design; this layout is ours.
//
// k_pipe advances two to four time steps per launch with the intermediate
// populations kept in LDS, so the populations cross HBM once per launch;
// k_batch_step and k_batch_pipe run many lattices from one work list.
// All kernels share the node arithmetic below and give identical bits.
//
// Storage: FP64 populations, or deviations s_a = f_a - w_a rho_ref in FP32 /
// FP16 with FP32 collision arithmetic, or FP32 deviations with FP64
// collision arithmetic.  The EOS, psi and force stencil are always evaluated
// in FP64.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "host_layout.hpp"  // Item

namespace lbm {

constexpr int LMAX = 128;  // largest chunk height (rows) k_step marches (halo arrays in LDS)

// Constants of the MRT collision: rates s of the energy (e), energy-square (eps),
// energy-flux (q) and stress (n, 1/tau) moments over the squared row norms, h = 1
// - s/2, and sigma / (1/s - 1/2) of the improved scheme.
struct MrtDev {
  double e, eS, sig_e;      // -s_e/36, 6 h_e/36
  double p, pS, sig_eps;    // -s_eps/36, -6 h_eps/36
  double qa, qaF, qd, qdF;  // s_q/6, (1 + h_q)/6, -s_q/12, 1/6 - h_q/12
  double n, nxx, nxy;       // -s_n/4, h_n/2, h_n/4
};

// Per-lattice constants, prepared on the host.
struct RunDev {
  int32_t nx, ny, pitch, eos;
  int64_t plane;            // elements between direction a and a+1 at one node
  int64_t rs;               // elements between row y and y+1 of one direction
  int64_t elems;            // elements of the lattice's population buffer
  int64_t off;              // element offset of this lattice in the population pool
  double RT, c1, c2;        // EOS constants (see EosConst)
  double two_over_G, mG;    // 2/G and -G
  double inv_tau;
  // forcing scheme in general form: u_eq = u + c_eq F/rho,
  // F_a = w_a [3 Be e.F + Ce (9 (e.vf)(e.F) - 3 vf.F)], vf = u + c_f F/rho + sig F/psi^2
  double c_eq, c_f, sig, Ce;
  // products used by the collision with om = 1/tau and w0, w1, w2 = 4/9, 1/9, 1/36: om w0,
  // om w1, om w2, 1 - om; of collide: c_d = c_f - c_eq, om/2, om/3, Be/3; of
  // collide_pairs: w0 Ce, w1 Ce, w2 Ce, 3 w1 Be, 3 w2 Be, 3 om w1, 3 om w2
  double om_w0, om_w1, om_w2, om1;
  double c_d, om_2, om_3, Be_3;
  double wCe0, wCe1, wCe2, wBe3_1, wBe3_2, om_3w1, om_3w2;
  double rho_ref;           // deviation reference density (0 for FP64 storage)
  int32_t run;
  int32_t mrt;              // 1: multiple-relaxation-time collision (collide_mrt with m)
  MrtDev m;
};


// Balanced schedule of a batch: the rows of all strips laid end to end, every strip
// but the first preceded by `fill` units (what starting a piece costs in rows), are split
// evenly over the grid; block t (XCD-remapped) marches its share, one piece per item it
// overlaps (at most `cap` rows per piece), and calls piece(item, first row in the item,
// rows).
template <class Piece>
__device__ __forceinline__ void balanced_pieces(const Item* __restrict__ items, int nitems, int total,
                                                int t, int cap, int fill, Piece&& piece) {
  const int64_t len = (int64_t)total + (int64_t)fill * (nitems - 1);
  int64_t v = len * t / gridDim.x + fill;
  const int64_t e = len * (t + 1) / gridDim.x + fill;
  // item k: its fill units begin at row0 + k fill, its rows `fill` later
  auto start = [&](int k) { return (int64_t)items[k].row0 + (int64_t)k * fill; };
  int lo = 0, hi = nitems - 1;  // last item that begins at or before v
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start(mid) <= v) lo = mid;
    else hi = mid - 1;
  }
  for (int i = lo; v < e && i < nitems;) {
    const Item it = items[i];
    const int64_t base = start(i) + fill;
    v = max(v, base);
    const int y = (int)(v - base);
    const int n = (int)min(min(e - v, (int64_t)(it.nrows - y)), (int64_t)cap);
    if (n > 0) {
      piece(it, y, n);
      v += n;
    }
    if (v >= base + it.nrows) ++i;
  }
}

// List schedule of a batch: entry b of the list is block b's first item and its row0 that
// item's place among the items behind the gridDim + 1 entries (layout::add_heads), so that a
// block that has one item reads no second entry.  Sweep of 256 runs, FP16, us per step, with
// two dependent loads (place, then item) and with one: 2 x 4 24.9 and 21.7, 8 x 16 33.7 and
// 30.8; other types the same.
template <class Piece>
__device__ __forceinline__ void listed_pieces(const Item* __restrict__ list, Piece&& piece) {
  const Item* __restrict__ items = list + gridDim.x + 1;
  Item it = list[blockIdx.x];
  const int hi = list[blockIdx.x + 1].row0;
  for (int i = it.row0; i < hi;) {
    piece(it, 0, it.nrows);
    if (++i < hi) it = items[i];
  }
}

// Storage traits: E = element type in memory, R = collision arithmetic type;
// round(v) = the value a store followed by a load would give.  Cache policy
// per type, measured on the 4096 x 4096 droplet workload with two steps per
// launch: FP64 populations stream with non-temporal loads and stores (plain
// stores cost 10 %); FP32 deviations use plain loads and stores (9 % faster
// than non-temporal); FP32 storage with FP64 arithmetic and FP16 deviations
// show no difference.
struct f32s_f64a {};  // FP32 deviation storage with FP64 collision arithmetic
template <typename S> struct Store;
// E: stored type; R: collision arithmetic; P: type of psi, of the force and of
// the density they are evaluated at (FP64 for every storage type: the EOS and
// psi stay FP64 in the reduced-precision forms).  kConserve: after the FP32
// collision, restore the node's mass and momentum change exactly (see
// conserve()).  kPairs: BGK collision by pairs of directions (collide_pairs).  kDev: values are deviations from w_a rho_ref.
template <> struct Store<double> {
  using E = double;
  using R = double;
  using P = double;
  static constexpr bool kConserve = false;
  static constexpr bool kPairs = false;
  static constexpr bool kDev = false;
  static __device__ __forceinline__ R ld(const E* p) { return __builtin_nontemporal_load(p); }
  static __device__ __forceinline__ void st(E* p, R v) { __builtin_nontemporal_store(v, p); }
  static __device__ __forceinline__ R round(R v) { return v; }
};
template <> struct Store<float> {
  using E = float;
  using R = float;
  using P = double;
  static constexpr bool kConserve = true;
  static constexpr bool kPairs = false;
  static constexpr bool kDev = true;
  static __device__ __forceinline__ R ld(const E* p) { return *p; }
  static __device__ __forceinline__ void st(E* p, R v) { *p = v; }
  static __device__ __forceinline__ R round(R v) { return v; }
};
template <> struct Store<f32s_f64a> {
  using E = float;
  using R = double;
  using P = double;
  static constexpr bool kConserve = false;
  static constexpr bool kPairs = false;
  static constexpr bool kDev = true;
  static __device__ __forceinline__ R ld(const E* p) { return double(__builtin_nontemporal_load(p)); }
  static __device__ __forceinline__ void st(E* p, R v) { __builtin_nontemporal_store(float(v), p); }
  static __device__ __forceinline__ R round(R v) { return double(float(v)); }
};
template <> struct Store<__half> {
  using E = __half;
  using R = float;
  using P = double;
  static constexpr bool kConserve = false;
  static constexpr bool kPairs = true;
  static constexpr bool kDev = true;
  // The narrowing to FP16 takes its operand through an empty asm statement:
  // the backend otherwise folds it into the FMA that produced the operand (a
  // mixed-precision FMA with an FP16 result, one rounding instead of two) at
  // some call sites only, whatever the contraction setting, which breaks the
  // bitwise identity of the one- and multi-step kernels.
  static __device__ __forceinline__ _Float16 narrow(R v) {
    asm("" : "+v"(v));
    return static_cast<_Float16>(v);
  }
  static __device__ __forceinline__ R ld(const E* p) { return __half2float(*p); }
  static __device__ __forceinline__ void st(E* p, R v) {
    __half_raw h;
    h.data = narrow(v);
    *p = h;
  }
  static __device__ __forceinline__ R round(R v) { return static_cast<float>(narrow(v)); }
};

// Index-checked build (LBM_CHECK_INDEX): every global load and store of the
// step, copy and mass kernels checks its element offset against the lattice's
// buffer, and every tile its shape against the kernel's limits; a violation
// is counted in g_index_faults (read by lbm_debug_index_faults) and the access
// is skipped.  Release builds compile none of this.
#ifdef LBM_CHECK_INDEX
__device__ unsigned long long g_index_faults;
__device__ __forceinline__ bool index_ok(int64_t off, int64_t n) {
  if (off >= 0 && off < n) return true;
  atomicAdd(&g_index_faults, 1ull);
  return false;
}
#define LBM_TILE_CHECK(cond)                            \
  do {                                                  \
    if (!(cond)) atomicAdd(&g_index_faults, 1ull);      \
  } while (0)
#else
__device__ __forceinline__ bool index_ok(int64_t, int64_t) { return true; }
#define LBM_TILE_CHECK(cond) \
  do {                       \
  } while (0)
#endif

// D2Q9 directions e0=(0,0), e1=(1,0), e2=(0,1), e3=(-1,0), e4=(0,-1), e5=(1,1),
// e6=(-1,1), e7=(-1,-1), e8=(1,-1) (pull9, collide and the moments use this
// numbering); weights of Eq. (2):
__device__ constexpr double kW[9] = {4.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0,
                                     1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};

// Reciprocals: the hardware estimate (relative error below 2^-24, measured over
// 1e-9 .. 1e9) refined by one third-order step, r (1 + e + e^2) with e = 1 - x r
// (FP64; the truncation e^3 is below 2^-72, so about 1 ulp; one operation less
// than two Newton steps), or the single-precision estimate (FP32 arithmetic
// paths, 1 ulp).  Arguments are positive normal numbers (or non-finite in a
// diverged state).
__device__ __forceinline__ double rcp(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Column indices of one thread: its own column and the periodic neighbours.
struct Cols {
  unsigned x, xm, xp;
};
__device__ __forceinline__ Cols cols_of(int x, int nx) {
  return Cols{(unsigned)x, (unsigned)(x == 0 ? nx - 1 : x - 1), (unsigned)(x == nx - 1 ? 0 : x + 1)};
}

// Pull the 9 populations of node (c.x, y) from the post-collision field.  Row
// and plane offsets are uniform across the block (scalar registers); only the
// 32-bit column index varies per lane.
template <typename S>
__device__ __forceinline__ void pull9(const typename Store<S>::E* __restrict__ src, const RunDev& d,
                                      const Cols& c, int y, typename Store<S>::R (&f)[9]) {
  const int ym = y == 0 ? d.ny - 1 : y - 1;
  const int yp = y == d.ny - 1 ? 0 : y + 1;
  const int64_t P = d.plane;
  using T = Store<S>;
  const typename T::E* r0 = src + (int64_t)y * d.rs;
  const typename T::E* rm = src + (int64_t)ym * d.rs;
  const typename T::E* rp = src + (int64_t)yp * d.rs;
#ifdef LBM_CHECK_INDEX
  const typename T::E* p9[9] = {r0 + c.x,         r0 + P + c.xm,     rm + 2 * P + c.x,
                                r0 + 3 * P + c.xp, rp + 4 * P + c.x,  rm + 5 * P + c.xm,
                                rm + 6 * P + c.xp, rp + 7 * P + c.xp, rp + 8 * P + c.xm};
  for (int a = 0; a < 9; ++a) f[a] = index_ok(p9[a] - src, d.elems) ? T::ld(p9[a]) : typename T::R(0);
#else
  f[0] = T::ld(r0 + c.x);
  f[1] = T::ld(r0 + P + c.xm);
  f[2] = T::ld(rm + 2 * P + c.x);
  f[3] = T::ld(r0 + 3 * P + c.xp);
  f[4] = T::ld(rp + 4 * P + c.x);
  f[5] = T::ld(rm + 5 * P + c.xm);
  f[6] = T::ld(rm + 6 * P + c.xp);
  f[7] = T::ld(rp + 7 * P + c.xp);
  f[8] = T::ld(rp + 8 * P + c.xm);
#endif
}

// The arithmetic of one node update below is written with explicit fma()
// where a fused multiply-add is wanted and compiled with contraction off, so
// every kernel that inlines it performs the same operations and rounds the
// same way (the single-step, multi-step and batched kernels give identical bits).

// Density deviation sum_a s_a in the arithmetic type (pairwise order).
template <typename R>
__device__ __forceinline__ R sum9(const R (&s)[9]) {
#pragma clang fp contract(off)
  return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])) + s[8];
}

// psi^2 = 2 (p_EOS(rho) - rho/3) / G (Eq. 8 with Eq. 23 or Peng-Robinson).
__device__ __forceinline__ double psi2_of(double rho, const RunDev& d) {
#pragma clang fp contract(off)
  double p;
  if (d.eos == 0) {
    // rho RT (1 + e + e^2 - e^3)/(1 - e)^3 - c2 rho^2, e = b rho / 4
    const double e = d.c1 * rho, m = 1.0 - e;
    const double poly = fma(e, fma(e, m, 1.0), 1.0);
    p = fma((rho * d.RT) * poly, rcp((m * m) * m), -((d.c2 * rho) * rho));
  } else {
    // rho RT/(1 - b) - c2 rho^2/(1 + b(2 - b)) over one common reciprocal
    const double b = d.c1 * rho;
    const double q1 = 1.0 - b, q2 = fma(b, 2.0 - b, 1.0);
    p = fma(rho * d.RT, q2, -(((d.c2 * rho) * rho) * q1)) * rcp(q1 * q2);
  }
  return fma(rho, -1.0 / 3.0, p) * d.two_over_G;
}

// The correctly rounded square root of x > 0 and, in r, 1/sqrt(x) to 1-2 ulp, from one
// hardware reciprocal square root y (relative error below 2^-24): with e = 1 - x y^2,
// 1/sqrt(x) = r = y (1 + e/2 + 3 e^2/8 + ...), g = x r, and the root is g + (x - g^2) r/2.
// Before its rounding that is within 2^-50 ulp of the root; the 365 arguments of two binades
// whose root lies within 2^-46 ulp of a midpoint of two doubles were enumerated and all give
// the result of sqrt() (as do 2^30 random ones).  No scaling and no special cases: 9
// operations where sqrt() takes 17.  Not a number for x = 0, infinite or negative: a node
// with such a psi^2 has diverged.
__device__ __forceinline__ double root_of(double x, double& r) {
#pragma clang fp contract(off)
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  r = fma(y, e * fma(0.375, e, 0.5), y);
  const double g = x * r;
  return fma(fma(-g, g, x), 0.5 * r, g);
}
// 1/psi^2 from x = psi^2 and r = 1/psi: the square of r and one Newton step (error as the
// reciprocal's), or the single-precision estimate (FP32 arithmetic).
template <typename R> __device__ __forceinline__ R inverse_of(double x, double r) {
#pragma clang fp contract(off)
  if constexpr (std::is_same<R, float>::value) {
    return rcp(float(x));
  } else {
    const double c = r * r;
    return fma(c, fma(-x, c, 1.0), c);
  }
}

__device__ __forceinline__ double pressure_of(double rho, const RunDev& d) {
  if (d.eos == 0) {
    const double e = d.c1 * rho, m = 1.0 - e;
    return rho * d.RT * (1.0 + e * (1.0 + e * (1.0 - e))) / (m * m * m) - d.c2 * rho * rho;
  }
  return rho * d.RT / (1.0 - d.c1 * rho) - d.c2 * rho * rho / (1.0 + d.c1 * rho * (2.0 - d.c1 * rho));
}

// Interaction force of Eq. (3), w(1) = 1/3, w(2) = 1/12, from three psi rows (s = y-1, c
// = y, n = y+1; index i = x).
__device__ __forceinline__ void force3x3(const double* rs, const double* rc, const double* rn, int i,
                                         double mG, double& Fx, double& Fy) {
#pragma clang fp contract(off)
  const double dNE = rn[i + 1] - rs[i - 1];  // psi(x+e5) - psi(x-e5)
  const double dNW = rn[i - 1] - rs[i + 1];  // psi(x+e6) - psi(x-e6)
  const double Sx = fma(1.0 / 3.0, rc[i + 1] - rc[i - 1], (1.0 / 12.0) * (dNE - dNW));
  const double Sy = fma(1.0 / 3.0, rn[i] - rs[i], (1.0 / 12.0) * (dNE + dNW));
  const double c = mG * rc[i];
  Fx = c * Sx;
  Fy = c * Sy;
}

// BGK collision with the forcing scheme in general form (see RunDev).
//
// For direction a the update is s_a + om (seq_a - s_a) + F_a with
//   seq_a = w (drho + rho (3 e.u + 4.5 (e.u)^2 - 1.5 u.u))        (Eq. 2, deviation form)
//   F_a   = w [3 B_e e.F + C_e (9 (e.v)(e.F) - 3 v.F)]             (Eq. 12)
// The even part of om seq + F is om w drho and a quadratic form of e: with m = rho u_eq = j
// + c_eq F and the symmetric tensor (both terms already times w1 = 1/9)
//   T = om/2 m u + C_e v F,  S = T_xx + T_yy,
// it is -4/3 S, T_xx - S/3, T_yy - S/3 and S/6 +- T_xy/4 (1.5/4.5 = 3/9 = 1/3), and the odd
// part is q.e with q = om/3 m + B_e/3 F (over 4 for the diagonals).  Each pair of opposite
// directions is then s' = (1 - om) s + (P +- Q).  58 operations besides the moments and
// 1/rho, against 85 of collide_pairs, which evaluates (e.u)^2 and (e.v)(e.F) for each
// pair.  The density enters each P last, in one fma of its own: error of a node's update over
// w rho in FP64, mean and largest of 400,000 against quadruple precision: 0.98e-16 and
// 8.6e-16, collide_pairs 1.05e-16 and 1.05e-15 (FP32 1.65e-8, collide_pairs 1.79e-8).
template <typename R>
__device__ __forceinline__ void relax_pair(R& sa, R& sb, R P, R Q, R om1) {
#pragma clang fp contract(off)
  sa = fma(om1, sa, P + Q);
  sb = fma(om1, sb, P - Q);
}

template <typename R>
__device__ __forceinline__ void collide(R (&s)[9], R drho, R rho, R jx, R jy, R Fx, R Fy,
                                        R inv_psi2, const RunDev& d) {
#pragma clang fp contract(off)
  const R inv_rho = rcp(rho);
  const R mx = fma(R(d.c_eq), Fx, jx), my = fma(R(d.c_eq), Fy, jy);
  const R wx = mx * inv_rho, wy = my * inv_rho;
  const R k = fma(R(d.c_d), inv_rho, R(d.sig) * inv_psi2);
  const R vx = fma(k, Fx, wx), vy = fma(k, Fy, wy);
  const R om_2 = R(d.om_2), Ce = R(d.Ce), om1 = R(d.om1);
  const R ax = om_2 * mx, ay = om_2 * my, bx = Ce * Fx, by = Ce * Fy;
  const R Txx = fma(ax, wx, bx * vx), Tyy = fma(ay, wy, by * vy);
  const R Txy = fma(ax, wy, fma(ay, wx, fma(bx, vy, by * vx)));
  const R S = Txx + Tyy, S3 = R(-1.0 / 3.0) * S, S6 = R(1.0 / 6.0) * S;
  const R om_3 = R(d.om_3), Be_3 = R(d.Be_3);
  const R qx = fma(om_3, mx, Be_3 * Fx), qy = fma(om_3, my, Be_3 * Fy);
  const R w1 = R(d.om_w1), w2 = R(d.om_w2);
  s[0] = fma(om1, s[0], fma(R(d.om_w0), drho, R(4) * S3));
  // axis pairs (e1, e3 = -e1), (e2, e4 = -e2)
  relax_pair(s[1], s[3], fma(w1, drho, Txx + S3), qx, om1);
  relax_pair(s[2], s[4], fma(w1, drho, Tyy + S3), qy, om1);
  // diagonal pairs (e5 = (1,1), e7 = -e5), (e6 = (-1,1), e8 = -e6)
  relax_pair(s[5], s[7], fma(w2, drho, fma(R(0.25), Txy, S6)), R(0.25) * (qx + qy), om1);
  relax_pair(s[6], s[8], fma(w2, drho, fma(R(-0.25), Txy, S6)), R(0.25) * (qy - qx), om1);
}

// The same by pairs of directions, for FP16 storage: there a last-bit difference of an FP32
// result turns roundings to FP16, and this form gives the populations that FP16 lattices have
// always had, bit for bit.  With X = drho + rho (4.5 (e.u)^2 - 1.5 u.u), om seq = om w X +-
// 3 om w rho e.u and F_a = C +- D, s' = (1 - om) s + (P +- Q) with P = om w X + C, Q = 3 om w
// rho e.u + D (the products of om and the weights are per-lattice constants).
template <typename R>
__device__ __forceinline__ void collide_pair(R& sa, R& sb, R eu, R eF, R ev, R omw, R omwr3, R wCe,
                                             R wBe3, R rho, R drho, R usq, R vF3, R om1) {
#pragma clang fp contract(off)
  const R X = fma(rho, fma(R(4.5) * eu, eu, -usq), drho);
  const R C = wCe * fma(R(9) * ev, eF, -vF3);
  const R P = fma(omw, X, C);
  const R Q = fma(omwr3, eu, wBe3 * eF);
  sa = fma(om1, sa, P + Q);
  sb = fma(om1, sb, P - Q);
}

template <typename R>
__device__ __forceinline__ void collide_pairs(R (&s)[9], R drho, R rho, R jx, R jy, R Fx, R Fy,
                                              R inv_psi2, const RunDev& d) {
#pragma clang fp contract(off)
  const R inv_rho = rcp(rho);
  const R ux = jx * inv_rho, uy = jy * inv_rho;
  const R Fr_x = Fx * inv_rho, Fr_y = Fy * inv_rho;
  const R wx = fma(R(d.c_eq), Fr_x, ux), wy = fma(R(d.c_eq), Fr_y, uy);
  const R sg = R(d.sig) * inv_psi2;
  const R vx = fma(sg, Fx, fma(R(d.c_f), Fr_x, ux)), vy = fma(sg, Fy, fma(R(d.c_f), Fr_y, uy));
  const R om1 = R(d.om1);
  const R usq = R(1.5) * fma(wx, wx, wy * wy);
  const R vF3 = R(3) * fma(vx, Fx, vy * Fy);
  const R omw1 = R(d.om_w1), omw2 = R(d.om_w2);
  const R omwr3_1 = R(d.om_3w1) * rho, omwr3_2 = R(d.om_3w2) * rho;
  const R wCe1 = R(d.wCe1), wBe3_1 = R(d.wBe3_1), wCe2 = R(d.wCe2), wBe3_2 = R(d.wBe3_2);
  // rest direction: e = 0
  s[0] = fma(om1, s[0], fma(R(d.om_w0), fma(rho, -usq, drho), R(d.wCe0) * -vF3));
  // axis pairs (e1, e3 = -e1), (e2, e4 = -e2)
  collide_pair(s[1], s[3], wx, Fx, vx, omw1, omwr3_1, wCe1, wBe3_1, rho, drho, usq, vF3, om1);
  collide_pair(s[2], s[4], wy, Fy, vy, omw1, omwr3_1, wCe1, wBe3_1, rho, drho, usq, vF3, om1);
  // diagonal pairs (e5 = (1,1), e7 = -e5), (e6 = (-1,1), e8 = -e6)
  collide_pair(s[5], s[7], wx + wy, Fx + Fy, vx + vy, omw2, omwr3_2, wCe2, wBe3_2, rho, drho, usq,
               vF3, om1);
  collide_pair(s[6], s[8], wy - wx, Fy - Fx, vy - vx, omw2, omwr3_2, wCe2, wBe3_2, rho, drho, usq,
               vF3, om1);
}

// Multiple-relaxation-time collision with the improved forcing scheme, on the
// D2Q9 moments of Lallemand and Luo (2000): rho, e, eps, j_x, q_x, j_y, q_y,
// p_xx, p_xy (squared row norms 9, 36, 36, 6, 12, 6, 12, 4, 4).  Each moment
// relaxes at its own rate toward the moments of the Eq. (2) equilibrium at
// v = u + F/(2 rho),
//   e_eq = rho(-2 + 3|v|^2), eps_eq = rho(1 - 3|v|^2), q_eq = -rho v,
//   p_xx,eq = rho(vx^2 - vy^2), p_xy,eq = rho vx vy,
// and receives (1 - s/2) times the moment of Eq. (31)'s bracket taken with the
// moment's own modified velocity v' = v + sigma F / ((1/s - 1/2) psi^2):
//   S_e = 6 v'.F, S_eps = -6 v'.F, S_q = -F, S_xx = 2(v'x Fx - v'y Fy), S_xy = v'x Fy + v'y Fx.
// The conserved moments need no relaxation: rho' = rho and j' = j + F (any
// momentum rate gives this).  In deviation storage the moments of w rho_ref,
// rho_ref (1, -2, 1, 0, ...), are taken out of rho, e and eps.  With every rate
// 1/tau this is the BGK update of collide() up to rounding.
//
// Only the changes of the moments go through the inverse transform, added to
// the populations as they are: with m = j + F/2 = rho v the changes over the
// row norms are r1 (e), r2 (eps), r7 (p_xx), r8 (p_xy), and the j and q changes
// enter the axis directions as ox, oy and the diagonal ones as X +- Y (per-lattice
// constants hold the rates over the norms, see MrtDev).
template <typename R>
__device__ __forceinline__ void collide_mrt(R (&s)[9], R drho, R rho, R jx, R jy, R Fx, R Fy,
                                            R inv_psi2, const RunDev& d) {
#pragma clang fp contract(off)
  const MrtDev& k = d.m;
  const R inv_rho = rcp(rho);
  const R mx = fma(R(0.5), Fx, jx), my = fma(R(0.5), Fy, jy);
  const R vx = mx * inv_rho, vy = my * inv_rho;
  const R w = fma(mx, vx, my * vy), vF = fma(vx, Fx, vy * Fy);  // rho |v|^2, v.F
  const R FF = fma(Fx, Fx, Fy * Fy) * inv_psi2;
  const R ax = s[1] + s[3], ay = s[2] + s[4], a = ax + ay;
  const R p57 = s[5] + s[7], p68 = s[6] + s[8], dg = p57 + p68;
  const R e = fma(R(-4), s[0], fma(R(2), dg, -a));
  const R ep = fma(R(4), s[0], fma(R(-2), a, dg));
  const R r1 = fma(R(k.e), fma(R(-3), w, fma(R(2), drho, e)), R(k.eS) * fma(R(k.sig_e), FF, vF));
  const R r2 = fma(R(k.p), fma(R(3), w, ep - drho), R(k.pS) * fma(R(k.sig_eps), FF, vF));
  // q + m = j - 3 (s1 - s3) + m, and likewise in y
  const R gx = fma(R(-3), s[1] - s[3], jx) + mx, gy = fma(R(-3), s[2] - s[4], jy) + my;
  const R ox = fma(R(k.qa), gx, R(k.qaF) * Fx), oy = fma(R(k.qa), gy, R(k.qaF) * Fy);
  const R X = fma(R(k.qd), gx, R(k.qdF) * Fx), Y = fma(R(k.qd), gy, R(k.qdF) * Fy);
  const R kn = R(d.sig) * inv_psi2;
  const R ux = fma(kn, Fx, vx), uy = fma(kn, Fy, vy);           // v' of the stress moments
  const R dxx = (ax - ay) - fma(mx, vx, -(my * vy)), dxy = fma(-mx, vy, p57 - p68);
  const R r7 = fma(R(k.n), dxx, R(k.nxx) * fma(ux, Fx, -(uy * Fy)));
  const R r8 = fma(R(k.n), dxy, R(k.nxy) * fma(ux, Fy, uy * Fx));
  s[0] = fma(R(4), r2 - r1, s[0]);
  const R A = fma(R(-2), r2, -r1), Dg = fma(R(2), r1, r2);
  const R Ap = A + r7, Am = A - r7, Dp = Dg + r8, Dm = Dg - r8, XpY = X + Y, XmY = X - Y;
  s[1] += Ap + ox;
  s[3] += Ap - ox;
  s[2] += Am + oy;
  s[4] += Am - oy;
  s[5] += Dp + XpY;
  s[7] += Dp - XpY;
  s[6] += Dm - XmY;
  s[8] += Dm + XmY;
}

template <typename R>
__device__ __forceinline__ R mom_x(const R (&s)[9]) {
  return ((s[1] - s[3]) + (s[5] - s[7])) + (s[8] - s[6]);
}
template <typename R>
__device__ __forceinline__ R mom_y(const R (&s)[9]) {
  return ((s[2] - s[4]) + (s[5] - s[7])) + (s[6] - s[8]);
}

// Momentum of FP32 values (as FP64 t) summed in FP64: exact unless the
// values span more than 29 binary orders of magnitude, and then wrong only by
// an FP64 rounding of the largest, far below an FP32 rounding; being exact,
// the sums do not depend on their order.
__device__ __forceinline__ void exact_momentum(const double (&t)[9], double& jx, double& jy) {
#pragma clang fp contract(off)
  const double u = t[5] - t[7], v = t[8] - t[6];
  jx = ((t[1] - t[3]) + u) + v;
  jy = ((t[2] - t[4]) + u) - v;
}
// Mass and momentum of nine FP32 values, exactly (as exact_momentum).
__device__ __forceinline__ void exact_moments(const float (&s)[9], double& m, double& jx, double& jy) {
#pragma clang fp contract(off)
  double t[9];
#pragma unroll
  for (int a = 0; a < 9; ++a) t[a] = double(s[a]);
  m = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7])) + t[8];
  exact_momentum(t, jx, jy);
}

// The collision conserves mass and changes the momentum by exactly F (every
// forcing scheme here, BGK or MRT).  In FP32 arithmetic each updated
// population carries its own rounding, and at a steady state the same
// roundings recur every step: a persistent mass and momentum source at every
// node that the slow bulk dynamics integrate into visibly shifted coexistence
// densities.  conserve() puts the momentum change of the new populations back
// to exactly F (half the x defect on e1 and -e1, likewise y on e2, -e4) and the
// mass back to exactly the old mass on the rest population, computed in FP64;
// what remains is one FP32 rounding of five values.
__device__ __forceinline__ void conserve(float (&s)[9], double m_t, double jx_t, double jy_t) {
#pragma clang fp contract(off)
  double t[9], jx, jy;
  t[0] = 0.0;  // the rest population carries no momentum
#pragma unroll
  for (int a = 1; a < 9; ++a) t[a] = double(s[a]);
  exact_momentum(t, jx, jy);
  const double dx = 0.5 * (jx_t - jx), dy = 0.5 * (jy_t - jy);
  s[1] = float(t[1] + dx);
  s[3] = float(t[3] - dx);
  s[2] = float(t[2] + dy);
  s[4] = float(t[4] - dy);
#pragma unroll
  for (int a = 1; a < 5; ++a) t[a] = double(s[a]);
  const double rest = ((t[1] + t[2]) + (t[3] + t[4])) + ((t[5] + t[6]) + (t[7] + t[8]));
  s[0] = float(m_t - rest);
}

// What a pulled row keeps for its collision: the summed stored values (the density
// or its deviation) and 1/psi^2.
template <typename S> struct NodeQ {
  typename Store<S>::R drho = 0, ip2 = 0;
};

// Density from the summed stored values.
template <typename S>
__device__ __forceinline__ double density(typename Store<S>::R drho, const RunDev& d) {
  if constexpr (Store<S>::kDev) return d.rho_ref + double(drho);
  return drho;
}

// psi of a pulled node; q receives what its collision needs.
template <typename S>
__device__ __forceinline__ double eval_psi(const typename Store<S>::R (&f)[9], const RunDev& d,
                                           NodeQ<S>& q) {
  using R = typename Store<S>::R;
  q.drho = sum9(f);
  const double psi2 = psi2_of(density<S>(q.drho, d), d);
  double r;
  const double psi = root_of(psi2, r);
  q.ip2 = inverse_of<R>(psi2, r);
  // sigma = 0 does not use it, and psi^2 may then lie outside the range of FP32
  if constexpr (std::is_same<R, float>::value) q.ip2 = d.sig != 0.0 ? q.ip2 : 0.0f;
  return psi;
}

// One node update: collision (BGK or MRT) of the pulled values f with the force
// (Fx, Fy) (FP64), for FP32 storage with conserve(); psi: the node's own.  True if the
// node is bad (density or psi^2 not positive, or not a number).
template <typename S, bool MRT>
__device__ __forceinline__ bool update_node(typename Store<S>::R (&f)[9], const NodeQ<S>& q, double psi,
                                            double Fx, double Fy, const RunDev& d) {
  using R = typename Store<S>::R;
  const double rho = density<S>(q.drho, d);
  auto collision = [&](R jx, R jy) __attribute__((always_inline)) {
    if constexpr (MRT)
      collide_mrt<R>(f, q.drho, R(rho), jx, jy, R(Fx), R(Fy), q.ip2, d);
    else if constexpr (Store<S>::kPairs)
      collide_pairs<R>(f, q.drho, R(rho), jx, jy, R(Fx), R(Fy), q.ip2, d);
    else
      collide<R>(f, q.drho, R(rho), jx, jy, R(Fx), R(Fy), q.ip2, d);
  };
  if constexpr (Store<S>::kConserve) {
    double m, jx, jy;
    exact_moments(f, m, jx, jy);
    collision(R(jx), R(jy));
    conserve(f, m, jx + Fx, jy + Fy);
  } else {
    collision(mom_x(f), mom_y(f));
  }
  return !(psi > 0.0) || !(rho > 0.0);
}

// Force and collision of a node from the psi rows around it; true if it is bad.
template <typename S, bool MRT>
__device__ __forceinline__ bool finish_node(typename Store<S>::R (&f)[9], const NodeQ<S>& q,
                                            const double* rs, const double* rc, const double* rn, int i,
                                            const RunDev& d) {
  double Fx, Fy;
  force3x3(rs, rc, rn, i, d.mG, Fx, Fy);
  return update_node<S, MRT>(f, q, rc[i], Fx, Fy, d);
}

// One tile: columns [x0, x0+ncols), rows [y0, y0+nrows), nrows <= LMAX.
// All threads of the block call it (barriers inside); ring is [4][SW+2],
// haloL/haloR [LMAX+2].  PF is the number of rows whose loads are in flight
// while a row is collided: with PF = 2 the loads of row y+2 are issued before
// the psi of row y+1 is evaluated and row y is collided.
template <typename S, int NW, int PF, bool MRT = false>
__device__ __forceinline__ void tile_step(const typename Store<S>::E* __restrict__ src,
                                          typename Store<S>::E* __restrict__ dst,
                                          const RunDev& d, int x0, int y0, int ncols, int nrows,
                                          unsigned long long step,
                                          unsigned long long* __restrict__ flag,
                                          typename Store<S>::P (*ring)[64 * NW + 2],
                                          typename Store<S>::P* haloL, typename Store<S>::P* haloR) {
  using T = Store<S>;
  using R = typename T::R;
  constexpr int SW = 64 * NW;
  const int tid = threadIdx.x;
  LBM_TILE_CHECK(ncols >= 1 && ncols <= SW && nrows >= 1 && nrows <= LMAX && x0 >= 0 &&
                 x0 + ncols <= d.nx && y0 >= 0 && y0 + nrows <= d.ny);
  const bool act = tid < ncols;
  const int x = x0 + tid;
  const Cols cx = cols_of(act ? x : x0, d.nx);
  const int xl = x0 == 0 ? d.nx - 1 : x0 - 1;
  const int xr = x0 + ncols >= d.nx ? 0 : x0 + ncols;
  bool bad = false;

  // preload rows y0-1 (ring slot 0) and y0 (slot 1); with PF = 2 also issue row
  // y0+1.  The loads are issued before the halo prologue so that both wait on
  // memory together.
  R fc[9], fn[9], fp[9];
  if (act) {
    pull9<S>(src, d, cx, y0 == 0 ? d.ny - 1 : y0 - 1, fp);
    pull9<S>(src, d, cx, y0, fc);
    if (PF == 2) pull9<S>(src, d, cx, y0 + 1 == d.ny ? 0 : y0 + 1, fn);
  }

  // prologue: psi of the two halo columns for rows y0-1 .. y0+nrows
  for (int i = tid; i < 2 * (nrows + 2); i += SW) {
    const int k = i >> 1;
    int yy = y0 - 1 + k;
    yy = yy < 0 ? yy + d.ny : (yy >= d.ny ? yy - d.ny : yy);
    R f[9];
    pull9<S>(src, d, cols_of((i & 1) ? xr : xl, d.nx), yy, f);
    NodeQ<S> q;
    ((i & 1) ? haloR : haloL)[k] = eval_psi<S>(f, d, q);
  }

  NodeQ<S> qc;
  if (act) {
    ring[0][tid + 1] = eval_psi<S>(fp, d, qc);
    ring[1][tid + 1] = eval_psi<S>(fc, d, qc);
  }
  __syncthreads();  // the halo columns are in LDS
  if (tid == 0) {
    ring[0][0] = haloL[0];
    ring[0][ncols + 1] = haloR[0];
    ring[1][0] = haloL[1];
    ring[1][ncols + 1] = haloR[1];
  }

  for (int j = 0; j < nrows; ++j) {
    const int y = y0 + j;
    const int yn = y + 1 == d.ny ? 0 : y + 1;
    const int sl = (j + 2) & 3;
    R fnn[9];
    NodeQ<S> qn;
    if (act) {
      if (PF == 2) {
        if (j + 1 < nrows) pull9<S>(src, d, cx, yn + 1 == d.ny ? 0 : yn + 1, fnn);
      } else {
        pull9<S>(src, d, cx, yn, fn);
      }
      ring[sl][tid + 1] = eval_psi<S>(fn, d, qn);
    }
    if (tid == 0) {
      ring[sl][0] = haloL[j + 2];
      ring[sl][ncols + 1] = haloR[j + 2];
    }
    __syncthreads();
    if (act) {
      bad |= finish_node<S, MRT>(fc, qc, ring[j & 3], ring[(j + 1) & 3], ring[sl], tid + 1, d);
      typename T::E* row = dst + (int64_t)y * d.rs;
#pragma unroll
      for (int a = 0; a < 9; ++a)
        if (index_ok(row + a * d.plane + cx.x - dst, d.elems)) T::st(row + a * d.plane + cx.x, fc[a]);
#pragma unroll
      for (int a = 0; a < 9; ++a) fc[a] = fn[a];
      qc = qn;
      if (PF == 2 && j + 1 < nrows) {
#pragma unroll
        for (int a = 0; a < 9; ++a) fn[a] = fnn[a];
      }
    }
  }
  // divergence: one atomic per wave that saw a bad node
  if (__ballot(bad) != 0 && __lane_id() == 0) atomicMin(flag, step);
}

// A run that diverged at an earlier launch is frozen: instead of a time step
// its tiles copy the stored populations unchanged from src to dst, so both
// buffers hold the state the diverging launch wrote, whatever the parity of
// later launches.  Columns [x0, x0+ncols), rows [y0, y0+nrows), SW threads.
template <typename S, int SW>
__device__ __forceinline__ void copy_tile(const typename Store<S>::E* __restrict__ src,
                                          typename Store<S>::E* __restrict__ dst, const RunDev& d,
                                          int x0, int y0, int ncols, int nrows) {
  if ((int)threadIdx.x >= ncols) return;
  const int x = x0 + (int)threadIdx.x;
  for (int j = 0; j < nrows; ++j) {
    const int64_t o = (int64_t)(y0 + j) * d.rs + x;
#pragma unroll
    for (int a = 0; a < 9; ++a)
      if (index_ok(o + a * d.plane, d.elems)) dst[o + a * d.plane] = src[o + a * d.plane];
  }
}

// XCD-aware block order: consecutive tiles go to the same XCD (blocks are
// dispatched round-robin over the 8 XCDs), so halo rows/columns shared by
// neighbouring tiles are found in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int n) {
  const int q = n >> 3, r = n & 7, k = b & 7, i = b >> 3;
  return k * q + (k < r ? k : r) + i;
}

// Single-lattice step.  L > 0: one block per (strip, L-row chunk).  L == 0:
// balanced schedule, the strip-major row space [0, nstrips*ny) is split evenly
// over the grid (sized to the resident capacity) and each block marches its
// share in pieces of at most LMAX rows.
template <typename S, int NW, int PF, bool MRT = false>
__global__ __launch_bounds__(64 * NW) void k_step(const typename Store<S>::E* __restrict__ src,
                                                  typename Store<S>::E* __restrict__ dst,
                                                  RunDev d, int L, int nstrips,
                                                  const unsigned long long* stepbase,
                                                  unsigned long long steplocal,
                                                  unsigned long long* flag) {
  __shared__ typename Store<S>::P ring[4][64 * NW + 2];
  __shared__ typename Store<S>::P haloL[LMAX + 2], haloR[LMAX + 2];
  constexpr int SW = 64 * NW;
  const unsigned long long step = (stepbase ? *stepbase : 0ull) + steplocal;
  const bool frozen = *flag < step;  // diverged at an earlier step
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  if (L > 0) {
    const int sy = t / nstrips, sx = t - sy * nstrips;
    const int x0 = sx * SW, y0 = sy * L;
    if (frozen)
      copy_tile<S, SW>(src, dst, d, x0, y0, min(SW, d.nx - x0), min(L, d.ny - y0));
    else
      tile_step<S, NW, PF, MRT>(src, dst, d, x0, y0, min(SW, d.nx - x0), min(L, d.ny - y0), step, flag,
                           ring, haloL, haloR);
    return;
  }
  const int64_t total = (int64_t)nstrips * d.ny;
  int64_t r = total * t / gridDim.x;
  const int64_t e = total * (t + 1) / gridDim.x;
  while (r < e) {
    const int s = (int)(r / d.ny), y = (int)(r - (int64_t)s * d.ny);
    int n = (int)min(e - r, (int64_t)(d.ny - y));
    n = min(n, LMAX);
    const int x0 = s * SW;
    if (frozen)
      copy_tile<S, SW>(src, dst, d, x0, y, min(SW, d.nx - x0), n);
    else
      tile_step<S, NW, PF, MRT>(src, dst, d, x0, y, min(SW, d.nx - x0), n, step, flag, ring, haloL,
                           haloR);
    r += n;
    __syncthreads();  // LDS is reused by the next piece
  }
}

// ---- several time steps per launch: one group of waves per step ------------------

// The populations cross HBM once per TS steps (TS = 2, 3 or 4).  A block is TS
// groups of NW waves; group l runs step l+1 of a strip of W = 64 NW columns, all
// groups marching up the rows together, each four rows behind the one before it,
// with one barrier per row.  In one march row a group
//   * pulls row p of its step: the first group from global memory (loaded one march
//     row ahead), the others from the exchange rows in LDS that the group before
//     them filled;
//   * evaluates psi of row p and leaves it in a ring of four rows in LDS;
//   * collides row p-2, whose psi rows the last three march rows left there, and hands the
//     result to the next group through the exchange rows; the last group stores it.
// Lane i owns column x0 - H + i, H = 2 TS - 1, in every step: step l is right on the
// lanes 2l .. and n0-1-2l (psi) and one lane further in (collision), so the last one
// is right on the ncols lanes from H on, and only those are stored.  The other
// lanes, rows outside a step's range and the first march rows compute values that
// no lane, row or step in range reads.  All steps use the arithmetic of single
// launches in the same order: bitwise equal.
//
// Why one group per step: a wave holds one step's rows only (145 VGPRs in FP64, 125
// with FP16 storage, against 254 for one wave doing three steps), so 3-4 waves per
// SIMD hide latency instead of 2, four steps fit where three did, and rows rotate by
// the names of unrolled registers and LDS slots instead of moves.  us per step, one wave
// for two or three steps -> one group per step, four steps: FP64 4096 x 4096 231 -> 143
// (4.8 TB/s counted; a plain copy gets 5.1), FP16 123 -> 93 (bound by vector issue), FP32
// 3000 x 2501 82 -> 59, FP32 with FP64 collide 1500 x 1001 27 -> 17, FP64 1024 x 1024 29
// -> 14.  A version with two barriers per row (collision after the exchange of the same
// row) took 1.2 times as long in FP64 and 1.55 times in FP16.  The figures that follow
// compare schedules and tiles with one another; the node arithmetic they were taken with was
// 4 to 10 % faster and less exact than this one.

// Barrier that orders LDS only: global loads and stores in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS of a block.  ex: the populations a step hands to the next.  A row collided in
// march row j leaves nine values: e4, e7, e8 are pulled one march row later (by the
// row below), e0, e1, e3 two and e2, e5, e6 three march rows later; a slot may be
// refilled one barrier after its last read, so they take 2, 4 (3 would do) and 4
// slots, j mod 4 with the loop unrolled by four.  The pads take the reads of lanes 0
// and W-1 past the ends (never used).
template <typename S, int W, int TS> struct PipeLds {
  double pad0[1];
  double psi[TS][4][W];  // psi of four march rows per step
  typename Store<S>::R ex[TS - 1][30][W];
  double pad1[1];
};
// FP64, three waves per step, four steps: 162,832 of the 163,840 bytes of a CU.
static_assert(sizeof(PipeLds<double, 192, 4>) <= 160 * 1024, "LDS of a CU");

// Byte offsets of one thread's columns in a row; nx * element size stays below 2^32
// (the launcher falls back to single steps otherwise).
struct ColBytes {
  unsigned x, xm, xp;
};
template <typename S>
__device__ __forceinline__ typename Store<S>::R ld_at(const char* p, unsigned off, const char* src,
                                                      const RunDev& d) {
  using E = typename Store<S>::E;
  const E* q = reinterpret_cast<const E*>(p + off);
  if (!index_ok(q - reinterpret_cast<const E*>(src), d.elems)) return typename Store<S>::R(0);
  return Store<S>::ld(q);
}
// pull9 of row y with its neighbour rows ym and yp given.
template <typename S>
__device__ __forceinline__ void pull9b(const char* src, const RunDev& d, const ColBytes& cb, int ym, int y,
                                       int yp, typename Store<S>::R (&f)[9]) {
  const int64_t P = d.plane * sizeof(typename Store<S>::E), rs = d.rs * sizeof(typename Store<S>::E);
  // opaque copies: the compiler otherwise widens the offsets once outside the row loop and
  // then adds a 64-bit address per lane and load
  ColBytes c;
  asm("" : "=v"(c.x) : "0"(cb.x));
  asm("" : "=v"(c.xm) : "0"(cb.xm));
  asm("" : "=v"(c.xp) : "0"(cb.xp));
  const char *r0 = src + (int64_t)y * rs, *rm = src + (int64_t)ym * rs, *rp = src + (int64_t)yp * rs;
  f[0] = ld_at<S>(r0, c.x, src, d);
  f[1] = ld_at<S>(r0 + P, c.xm, src, d);
  f[2] = ld_at<S>(rm + 2 * P, c.x, src, d);
  f[3] = ld_at<S>(r0 + 3 * P, c.xp, src, d);
  f[4] = ld_at<S>(rp + 4 * P, c.x, src, d);
  f[5] = ld_at<S>(rm + 5 * P, c.xm, src, d);
  f[6] = ld_at<S>(rm + 6 * P, c.xp, src, d);
  f[7] = ld_at<S>(rp + 7 * P, c.xp, src, d);
  f[8] = ld_at<S>(rp + 8 * P, c.xm, src, d);
}

// Exchange rows of march rows j with j mod 4 = K (x: the lane's entry of row 0): what a
// step leaves, rounded to the storage type, and what the next one pulls.
template <typename S, int W, int K>
__device__ __forceinline__ void pipe_push(typename Store<S>::R* x, const typename Store<S>::R (&f)[9]) {
  using T = Store<S>;
  constexpr int a1 = (K & 1) * 3, a2 = 6 + K * 3, a3 = 18 + K * 3;
  x[(a1 + 0) * W] = T::round(f[4]);
  x[(a1 + 1) * W] = T::round(f[7]);
  x[(a1 + 2) * W] = T::round(f[8]);
  x[(a2 + 0) * W] = T::round(f[0]);
  x[(a2 + 1) * W] = T::round(f[1]);
  x[(a2 + 2) * W] = T::round(f[3]);
  x[(a3 + 0) * W] = T::round(f[2]);
  x[(a3 + 1) * W] = T::round(f[5]);
  x[(a3 + 2) * W] = T::round(f[6]);
}
template <typename S, int W, int K>
__device__ __forceinline__ void pipe_pull(const typename Store<S>::R* x, typename Store<S>::R (&f)[9]) {
  constexpr int a1 = ((K + 1) & 1) * 3, a2 = 6 + ((K + 2) & 3) * 3, a3 = 18 + ((K + 1) & 3) * 3;
  f[4] = x[(a1 + 0) * W];
  f[7] = x[(a1 + 1) * W + 1];
  f[8] = x[(a1 + 2) * W - 1];
  f[0] = x[(a2 + 0) * W];
  f[1] = x[(a2 + 1) * W - 1];
  f[3] = x[(a2 + 2) * W + 1];
  f[2] = x[(a3 + 0) * W];
  f[5] = x[(a3 + 1) * W - 1];
  f[6] = x[(a3 + 2) * W + 1];
}

// A block's pieces follow one another without draining the pipeline: a group that has
// done its rows of a piece starts its rows of the next, while the groups behind it finish
// the last one.  Group l has rows jf .. je-1 of a piece's march rows, and the next piece's
// march row 0 is the one at which the first group is done, je of l = 0: no other group is
// busy with both (je of group l is at most (2l + 3) & ~3 later, its jf (6l) & ~3), and
// piece lengths are whole fours, so registers and LDS slots keep their rotation and a
// hand-over is never more than the 1-3 march rows apart that it is inside a piece.
// A sweep of 256 runs (3.1 million nodes, 2-3 pieces per block), us per launch of four
// steps, drained after each piece -> not: FP64 162 -> 158, FP32 with FP64 collide 153 ->
// 146, FP64 in chunks of 16 rows 216 -> 201.
// `owed`: barriers the group has yet to pass to reach the next piece's march row 0
// (negative: it is past it).
template <int TS> __device__ __forceinline__ void pipe_drain(int owed) {
  for (int k = -((2 * (TS - 1) + 3) & ~3); k < owed; ++k) lds_barrier();
}

// TS time steps of columns [x0, x0+ncols), rows [y0, y0+nrows); ncols <= W - 2H.  All
// threads of the block call it.  owed: 0 for a block's first piece, passed on from each
// piece to the next and to pipe_drain after the last.
template <typename S, int NW, int TS, bool MRT = false>
__device__ __forceinline__ void tile_pipe(const typename Store<S>::E* __restrict__ src,
                                          typename Store<S>::E* __restrict__ dst,
                                          const RunDev& d, int x0, int y0, int ncols, int nrows,
                                          unsigned long long step,
                                          unsigned long long* __restrict__ flag,
                                          PipeLds<S, 64 * NW, TS>& lds, int& owed) {
  using T = Store<S>;
  using E = typename T::E;
  using R = typename T::R;
  constexpr int W = 64 * NW, H = 2 * TS - 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lv = wave / NW;
  const int i = (wave - lv * NW) * 64 + (threadIdx.x & 63);
  LBM_TILE_CHECK(ncols >= 1 && ncols <= W - 2 * H && nrows >= 1 && x0 >= 0 && x0 + ncols <= d.nx &&
                 y0 >= 0 && y0 + nrows <= d.ny);
  const bool out = i >= H && i < ncols + H;
  int c = (x0 - H + min(i, ncols + 2 * H - 1)) % d.nx;
  if (c < 0) c += d.nx;
  double* const ps = &lds.psi[lv][0][0] + i;
  bool bad = false;
  // march rows of the first group, and of this step, widened to whole fours (the rows added
  // compute values that nothing reads)
  const int J = 4 * (TS - 1) + nrows + 3;
  const int jn = (J + 3) & ~3, jf = (6 * lv) & ~3, je = (J + 2 * lv + 3) & ~3;
  const int yc = y0 - H - 2 - 4 * lv;                  // row collided at march row j: yc + j
  auto in_rows = [&](int j) { return yc + j >= y0 && yc + j < y0 + nrows; };
  // rows p, p-1, p-2 and (first group) the one being loaded: buffer K = j mod 4 holds p,
  // K + 3 row p-1, K + 2 row p-2
  R F[4][9];
  double P[4] = {0, 0, 0, 0};
  NodeQ<S> Q[4];
  // psi of the pulled row to LDS (row K); collision of the row two below (buffer K + 2)
  // with the psi rows below (row K + 1), at and above it (row K + 3), which the last three
  // march rows left; row K held the one before those
  auto step_row = [&](auto kk) __attribute__((always_inline)) {
    constexpr int K = decltype(kk)::value, ks = (K + 1) & 3, kc = (K + 2) & 3, kn = (K + 3) & 3;
    const double *s = ps + ks * W, *c = ps + kc * W, *n = ps + kn * W;
    const double rs[3] = {s[-1], P[ks], s[1]}, rc[3] = {c[-1], P[kc], c[1]}, rn[3] = {n[-1], P[kn], n[1]};
    const bool b = finish_node<S, MRT>(F[kc], Q[kc], rs, rc, rn, 1, d);
    P[K] = eval_psi<S>(F[K], d, Q[K]);
    ps[K * W] = P[K];
    return b;
  };
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  using K3 = std::integral_constant<int, 3>;
  auto march = [&](auto&& row) __attribute__((always_inline)) {
    for (int j = -owed; j < jf; ++j) lds_barrier();
    for (int j = jf; j < je; j += 4) {
      row(j, K0{});
      row(j + 1, K1{});
      row(j + 2, K2{});
      row(j + 3, K3{});
    }
    owed = jn - je;
  };
  if (lv == 0) {
    R* xo = &lds.ex[0][0][0] + i;
    const char* sb = reinterpret_cast<const char*>(src);
    const ColBytes cb{(unsigned)(c * sizeof(E)), (unsigned)((c == 0 ? d.nx - 1 : c - 1) * sizeof(E)),
                      (unsigned)((c == d.nx - 1 ? 0 : c + 1) * sizeof(E))};
    auto next = [&](int v) { return v + 1 == d.ny ? 0 : v + 1; };
    int ym = (y0 - H - 1) % d.ny;
    if (ym < 0) ym += d.ny;
    int y = next(ym), yp = next(y);
    pull9b<S>(sb, d, cb, ym, y, yp, F[0]);
    auto row = [&](int j, auto kk) __attribute__((always_inline)) {
      constexpr int K = decltype(kk)::value;
      ym = y;
      y = yp;
      yp = next(yp);
      pull9b<S>(sb, d, cb, ym, y, yp, F[(K + 1) & 3]);
      bad |= step_row(kk) && out && in_rows(j);
      pipe_push<S, W, K>(xo, F[(K + 2) & 3]);
      lds_barrier();
    };
    march(row);
  } else if (lv < TS - 1) {
    const R* xi = &lds.ex[lv - 1][0][0] + i;
    R* xo = &lds.ex[lv < TS - 1 ? lv : 0][0][0] + i;
    auto row = [&](int j, auto kk) __attribute__((always_inline)) {
      constexpr int K = decltype(kk)::value;
      pipe_pull<S, W, K>(xi, F[K]);
      bad |= step_row(kk) && out && in_rows(j);
      pipe_push<S, W, K>(xo, F[(K + 2) & 3]);
      lds_barrier();
    };
    march(row);
  } else {
    const R* xi = &lds.ex[TS - 2][0][0] + i;
    const unsigned cb = (unsigned)(c * sizeof(E));
    auto row = [&](int j, auto kk) __attribute__((always_inline)) {
      constexpr int K = decltype(kk)::value;
      pipe_pull<S, W, K>(xi, F[K]);
      bad |= step_row(kk) && out && in_rows(j);
      if (out && in_rows(j)) {
        char* orow = reinterpret_cast<char*>(dst + (int64_t)(yc + j) * d.rs);
        unsigned co;
        asm("" : "=v"(co) : "0"(cb));
#pragma unroll
        for (int a = 0; a < 9; ++a) {
          E* q = reinterpret_cast<E*>(orow + a * d.plane * sizeof(E) + co);
          if (index_ok(q - dst, d.elems)) T::st(q, F[(K + 2) & 3][a]);
        }
      }
      lds_barrier();
    };
    march(row);
  }
  if (__ballot(bad) != 0 && __lane_id() == 0) atomicMin(flag, step + lv);
}

// Strip edges of the multi-step kernels are rounded down to multiples of this
// many columns (FP64: 8 columns = 64 B, so no 64-byte segment of a population
// row is written by two blocks).
template <typename S> struct StripAlign : std::integral_constant<int, 1> {};
template <> struct StripAlign<double> : std::integral_constant<int, 8> {};

// Waves per step of a multi-step tile: the strip class `waves` 4 (8 is the same) gives
// strips of 64 k columns less the halo with k = 4, or 3 with FP64 arithmetic (a CU's LDS
// holds four steps of 192 columns, not of 256, and three waves per SIMD have the registers
// that four have not; two steps of a single lattice may take six, see launch_pipe_s); 2
// gives the narrow ones, k = 2, for lattices that leave lanes of a wide strip idle.  FP32
// arithmetic is held to the 128 registers of four waves per SIMD: FP32 storage 4096 x 4096
// with k = 4 103 us per step, with k = 3 and 148 registers 110.
template <typename S> constexpr int pipe_nw(int waves) {
  return waves == 2 ? 2 : std::is_same<typename Store<S>::R, float>::value ? 4 : 3;
}
template <typename S> constexpr int pipe_waves_per_simd() {
  return std::is_same<typename Store<S>::R, float>::value ? 4 : 2;
}

// What a piece costs besides its rows, in rows: the first group's halo rows (pipe; a
// block's last piece takes pipe_drain_rows more), psi rows and the prologue (one-step
// kernels).
constexpr int pipe_fill(int ts) { return 4 * (ts - 1) + 3; }
constexpr int pipe_drain_rows(int ts) { return 2 * (ts - 1); }
constexpr int kStepFill = 3;

// Single lattice: strips of at most W - 2H columns spread evenly over nx.  L > 0: one
// block per (strip, L-row chunk).  L == 0: balanced schedule, every block marches one
// contiguous share of the strips laid end to end; a share is split where it crosses a
// strip boundary.
template <typename S, int NW, int TS, bool MRT = false>
__global__ __launch_bounds__(64 * NW * TS)
__attribute__((amdgpu_waves_per_eu(pipe_waves_per_simd<S>()))) void k_pipe(const typename Store<S>::E* __restrict__ src,
                                                       typename Store<S>::E* __restrict__ dst, RunDev d,
                                                       int L, int nstrips,
                                                       const unsigned long long* stepbase,
                                                       unsigned long long steplocal,
                                                       unsigned long long* flag) {
  __shared__ PipeLds<S, 64 * NW, TS> lds;
  const unsigned long long step = (stepbase ? *stepbase : 0ull) + steplocal;
  const bool frozen = *flag < step;  // diverged at an earlier step
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  auto edge = [&](int k) {
    constexpr int A = StripAlign<S>::value;
    return k >= nstrips ? d.nx : (int)((int64_t)k * d.nx / nstrips) / A * A;
  };
  int owed = 0;
  auto piece = [&](int s, int y, int n) {
    const int x0 = edge(s), nc = edge(s + 1) - x0;
    if (frozen)
      copy_tile<S, 64 * NW>(src, dst, d, x0, y, nc, n);
    else
      tile_pipe<S, NW, TS, MRT>(src, dst, d, x0, y, nc, n, step, flag, lds, owed);
  };
  if (L > 0) {
    const int sy = t / nstrips, s = t - sy * nstrips;
    piece(s, sy * L, min(L, d.ny - sy * L));
    pipe_drain<TS>(owed);
    return;
  }
  // Rows cost one each and every piece kFill more (the march rows that fill and drain
  // the pipeline), so shares are equal on a line on which every strip but the first is
  // preceded by kFill units, not in rows alone: a share that crosses into the next strip
  // pays for the second fill with fewer rows.  us per launch of four steps, equal rows ->
  // equal cost: 4096 x 4096 FP64 534 -> 529, 3000 x 2501 FP32 218 -> 207, 1500 x 1001 FP32
  // with FP64 collide 75 -> 63, 1024 x 1024 FP64 68 -> 55, 777 x 643 53 -> 39.
  constexpr int kFill = pipe_fill(TS);
  const int64_t per = (int64_t)d.ny + kFill, total = nstrips * per - kFill;
  auto at = [&](int k, int& s, int& y) {  // strip and row where share k begins
    const int64_t v = total * k / gridDim.x + kFill;
    s = (int)(v / per);
    y = max(0, (int)(v - s * per) - kFill);
  };
  int s, y, se, ye;
  at(t, s, y);
  at(t + 1, se, ye);  // the last share ends at (nstrips, 0)
  for (; s < se || (s == se && y < ye); ++s, y = 0) piece(s, y, (s < se ? d.ny : ye) - y);
  pipe_drain<TS>(owed);
}

// ---- small lattices: several steps of a patch, one node per thread ------------------

// pull9 of a row that differs from lane to lane.
template <typename S>
__device__ __forceinline__ void pull9_lane(const typename Store<S>::E* __restrict__ src, const RunDev& d,
                                           const Cols& c, int y, typename Store<S>::R (&f)[9]) {
  const int ym = y == 0 ? d.ny - 1 : y - 1, yp = y == d.ny - 1 ? 0 : y + 1;
  const int64_t P = d.plane, r0 = (int64_t)y * d.rs, rm = (int64_t)ym * d.rs, rp = (int64_t)yp * d.rs;
  const int64_t o[9] = {r0 + c.x,          r0 + P + c.xm,     rm + 2 * P + c.x,
                        r0 + 3 * P + c.xp, rp + 4 * P + c.x,  rm + 5 * P + c.xm,
                        rm + 6 * P + c.xp, rp + 7 * P + c.xp, rp + 8 * P + c.xm};
#pragma unroll
  for (int a = 0; a < 9; ++a)
    f[a] = index_ok(o[a], d.elems) ? Store<S>::ld(src + o[a]) : typename Store<S>::R(0);
}

// A block holds a patch of RX x RY nodes, a thread a node, and advances it TS steps on
// chip: every node pulls from global memory once, psi and the eight moving populations
// of each step go to the neighbours through LDS (two barriers per step), and the inner
// (RX - 2H) x (RY - 2H) nodes, H = 2 TS - 1, which the halo's wrong edge has not
// reached, are stored.  For lattices that leave most of the chip idle: a step there is
// latency (a launch, a load, two exchanges), and the march of the other kernels puts
// rows one after the other.  The recomputed halo costs 7.6 (22 x 22, four steps), 2.1 or
// 1.5 (32 x 32, three, two) times the work, so lattices that fill the chip take the pipe.
// The populations' loads go out before the divergence flag is waited for, which ends a
// chain of two latencies: 100 steps of 64 x 32 went from 194 to 188 us.
// us per step in a graph, FP64, best other tile -> patch: 64 x 32 4.3 -> 1.6, 128 x 64 4.4
// -> 1.7, 200 x 150 5.0 -> 2.6, 300 x 300 6.3 -> 3.5, 512 x 512 7.4 -> 7.4, 777 x 643 9.5
// -> 12.8.  Same arithmetic in the same order as single steps: bitwise equal.
template <typename S, int RX, int RY, int TS, bool MRT = false>
__global__ __launch_bounds__((RX * RY + 63) / 64 * 64) void k_patch(
    const typename Store<S>::E* __restrict__ src, typename Store<S>::E* __restrict__ dst, RunDev d, int ntx,
    const unsigned long long* stepbase, unsigned long long steplocal, unsigned long long* flag) {
  using T = Store<S>;
  using R = typename T::R;
  constexpr int H = 2 * TS - 1, TX = RX - 2 * H, TY = RY - 2 * H, N = RX * RY, PAD = RX + 1;
  __shared__ double psi[N + 2 * PAD];
  __shared__ R ex[TS > 1 ? 8 : 1][N + 2 * PAD];
  const int ty = blockIdx.x / ntx, tx = blockIdx.x - ty * ntx;
  const int i = min((int)threadIdx.x, N - 1);  // the last wave's idle lanes repeat a node
  const int ry = i / RX, rx = i - ry * RX;
  const int gx = tx * TX + rx - H, gy = ty * TY + ry - H;
  const bool out = threadIdx.x < N && rx >= H && rx < RX - H && ry >= H && ry < RY - H && gx < d.nx && gy < d.ny;
  // periodic image of column or row g of n, for g in (-w, n + w)
  auto wrap = [](int g, int n, int w) {
    if (n < w) {  // a patch wider than the lattice
      g %= n;
      return g < 0 ? g + n : g;
    }
    return g < 0 ? g + n : (g >= n ? g - n : g);
  };
  const int x = wrap(gx, d.nx, RX), y = wrap(gy, d.ny, RY);
  const Cols cx = cols_of(x, d.nx);
  // the node's populations are under way before the divergence flag is waited for
  R f[9];
  pull9_lane<S>(src, d, cx, y, f);
  const unsigned long long step = (stepbase ? *stepbase : 0ull) + steplocal;
  if (*flag < step) {  // diverged at an earlier step: frozen
    if (out) {
#pragma unroll
      for (int a = 0; a < 9; ++a) {
        const int64_t o = (int64_t)y * d.rs + a * d.plane + x;
        if (index_ok(o, d.elems)) dst[o] = src[o];
      }
    }
    return;
  }
  double* ps = psi + PAD + i;
  bool bad = false;
  int first = TS;
#pragma unroll
  for (int l = 0; l < TS; ++l) {
    NodeQ<S> q;
    *ps = eval_psi<S>(f, d, q);
    lds_barrier();
    const bool b = finish_node<S, MRT>(f, q, ps - RX, ps, ps + RX, 0, d);
    if (b && out && !bad) first = l;
    bad |= b && out;
    if (l < TS - 1) {
      R(*e)[N + 2 * PAD] = ex;
      const int k = PAD + i;
#pragma unroll
      for (int a = 1; a < 9; ++a) e[a - 1][k] = T::round(f[a]);
      f[0] = T::round(f[0]);
      lds_barrier();
      f[1] = e[0][k - 1];
      f[2] = e[1][k - RX];
      f[3] = e[2][k + 1];
      f[4] = e[3][k + RX];
      f[5] = e[4][k - RX - 1];
      f[6] = e[5][k - RX + 1];
      f[7] = e[6][k + RX + 1];
      f[8] = e[7][k + RX - 1];
    }
  }
  if (out) {
#pragma unroll
    for (int a = 0; a < 9; ++a) {
      const int64_t o = (int64_t)y * d.rs + a * d.plane + x;
      if (index_ok(o, d.elems)) T::st(dst + o, f[a]);
    }
  }
  if (bad) atomicMin(flag, step + first);
}

// Persistent batched step over a work list (listed_pieces, or balanced_pieces where
// total > 0).  A run frozen by divergence at an earlier launch is copied unchanged.
template <typename S, int NW, int PF, bool MRT = false>
__global__ __launch_bounds__(64 * NW) void k_batch_step(const typename Store<S>::E* __restrict__ src,
                                                        typename Store<S>::E* __restrict__ dst,
                                                        const RunDev* __restrict__ runs,
                                                        const Item* __restrict__ items, int nitems,
                                                        int total,
                                                        const unsigned long long* stepbase,
                                                        unsigned long long steplocal,
                                                        unsigned long long* flags) {
  __shared__ typename Store<S>::P ring[4][64 * NW + 2];
  __shared__ typename Store<S>::P haloL[LMAX + 2], haloR[LMAX + 2];
  const unsigned long long step = (stepbase ? *stepbase : 0ull) + steplocal;
  auto piece = [&](const Item& it, int y, int n) {
    const RunDev d = runs[it.run];
    if (flags[it.run] < step)  // frozen run
      copy_tile<S, 64 * NW>(src + d.off, dst + d.off, d, it.x0, it.y0 + y, it.ncols, n);
    else
      tile_step<S, NW, PF, MRT>(src + d.off, dst + d.off, d, it.x0, it.y0 + y, it.ncols, n, step,
                                &flags[it.run], ring, haloL, haloR);
    __syncthreads();  // LDS is reused by the next piece
  };
  if (total > 0)  // equal rows: counting kStepFill rows for a start was slower (FP64 1 x 0 66.4 -> 69.9)
    balanced_pieces(items, nitems, total, xcd_remap(blockIdx.x, gridDim.x), LMAX, 0, piece);
  else
    listed_pieces(items, piece);
}

// Persistent batched launch of TS steps (tile_pipe); the items are at most W - 2H columns
// wide.
template <typename S, int NW, int TS, bool MRT = false>
__global__ __launch_bounds__(64 * NW * TS)
__attribute__((amdgpu_waves_per_eu(pipe_waves_per_simd<S>()))) void k_batch_pipe(const typename Store<S>::E* __restrict__ src,
                                                             typename Store<S>::E* __restrict__ dst,
                                                             const RunDev* __restrict__ runs,
                                                             const Item* __restrict__ items, int nitems,
                                                             int total,
                                                             const unsigned long long* stepbase,
                                                             unsigned long long steplocal,
                                                             unsigned long long* flags) {
  __shared__ PipeLds<S, 64 * NW, TS> lds;
  const unsigned long long step = (stepbase ? *stepbase : 0ull) + steplocal;
  int owed = 0;
  auto piece = [&](const Item& it, int y, int n) {
    const RunDev d = runs[it.run];
    if (flags[it.run] < step)  // frozen run
      copy_tile<S, 64 * NW>(src + d.off, dst + d.off, d, it.x0, it.y0 + y, it.ncols, n);
    else
      tile_pipe<S, NW, TS, MRT>(src + d.off, dst + d.off, d, it.x0, it.y0 + y, it.ncols, n, step,
                                &flags[it.run], lds, owed);
  };
  if (total > 0)  // no row cap: no per-row arrays
    balanced_pieces(items, nitems, total, xcd_remap(blockIdx.x, gridDim.x), 1 << 30, pipe_fill(TS), piece);
  else
    listed_pieces(items, piece);
  pipe_drain<TS>(owed);
}

// Coexistence densities of flat interfaces with normal x, for every run of a
// batch: out[2r] = mean over y of rho at column nx/2 (liquid), out[2r+1] = the
// same at column 0 (vapour), in FP64 with rho decoded as the step kernels do
// (rho_ref + sum of the pulled populations).  One block per run; per-thread
// partial sums over rows tid, tid+256, ... then a fixed-order tree, so the
// result does not depend on timing.  A diverged run gives NaN.
template <typename S>
__global__ __launch_bounds__(256) void k_batch_coex(const typename Store<S>::E* __restrict__ pool,
                                                    const RunDev* __restrict__ runs,
                                                    const unsigned long long* __restrict__ flags,
                                                    double* __restrict__ out) {
  using R = typename Store<S>::R;
  __shared__ double sl[256], sg[256];
  const int r = blockIdx.x;
  const RunDev d = runs[r];
  const typename Store<S>::E* src = pool + d.off;
  const Cols cl = cols_of(d.nx / 2, d.nx), cg = cols_of(0, d.nx);
  double al = 0.0, ag = 0.0;
  for (int y = threadIdx.x; y < d.ny; y += 256) {
    R f[9];
    pull9<S>(src, d, cl, y, f);
    al += d.rho_ref + double(sum9(f));
    pull9<S>(src, d, cg, y, f);
    ag += d.rho_ref + double(sum9(f));
  }
  sl[threadIdx.x] = al;
  sg[threadIdx.x] = ag;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) {
      sl[threadIdx.x] += sl[threadIdx.x + k];
      sg[threadIdx.x] += sg[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const bool div = flags[r] != ~0ull;
    out[2 * r] = div ? __builtin_nan("") : sl[0] / d.ny;
    out[2 * r + 1] = div ? __builtin_nan("") : sg[0] / d.ny;
  }
}

// Graph helper: advance the device step counter after k steps.
__global__ void k_counter_add(unsigned long long* ctr, unsigned long long k) { *ctr += k; }
__global__ void k_counter_set(unsigned long long* ctr, unsigned long long v) { *ctr = v; }

// ---- diagnostics -------------------------------------------------------------

// Macroscopic fields: rho, v = u + F/(2 rho) (Table I, actual velocity) and p =
// p_EOS(rho).  One pass: a block of T threads (at most 256) owns up to T - 2 columns (a
// lane more on either side evaluates psi) and marches up a chunk of rows, the next row's loads in
// flight; psi goes to the neighbour lanes through a ring of four rows in LDS, one barrier per
// row.  Bound by memory: every population
// read once, four planes written once.  2048 x 2048 FP64 (302 + 134 MB): 98 us, 4.4
// TB/s, against 113 in two passes with psi and u going through memory.
template <typename S>
__global__ __launch_bounds__(256) void k_fields(const typename Store<S>::E* __restrict__ src, RunDev d, int L,
                                                int nstrips, double* __restrict__ rho_o,
                                                double* __restrict__ vx_o, double* __restrict__ vy_o,
                                                double* __restrict__ p_o) {
  using R = typename Store<S>::R;
  __shared__ double ring[4][256 + 2];
  const int tid = threadIdx.x;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int sy = t / nstrips, s = t - sy * nstrips;
  const int cols = blockDim.x - 2, x0 = s * cols, nc = min(cols, d.nx - x0);
  const int y0 = (int)((int64_t)sy * L), n = min(L, d.ny - y0);
  const bool out = tid >= 1 && tid <= nc;
  int x = x0 - 1 + min(tid, nc + 1);
  x = x < 0 ? x + d.nx : (x >= d.nx ? x - d.nx : x);
  const Cols cx = cols_of(x, d.nx);
  auto next = [&](int y) { return y + 1 == d.ny ? 0 : y + 1; };
  double rc = 0;  // rho and momentum of row p-1
  R jxc = 0, jyc = 0;
  R f[9], g[9];
  int y = y0 == 0 ? d.ny - 1 : y0 - 1;
  pull9<S>(src, d, cx, y, f);
  for (int j = 0; j < n + 2; ++j) {  // pulls row p = y0 - 1 + j, writes row p - 1
    y = next(y);
    if (j + 1 < n + 2) pull9<S>(src, d, cx, y, g);
    const R drho = sum9(f);
    const R jx = mom_x(f), jy = mom_y(f);
    const double r = density<S>(drho, d);
    ring[j & 3][tid + 1] = sqrt(psi2_of(r, d));  // 0 at an empty node, unlike root_of
    __syncthreads();
    if (j >= 2 && out) {
      double Fx, Fy;
      force3x3(ring[(j + 2) & 3], ring[(j + 3) & 3], ring[j & 3], tid + 1, d.mG, Fx, Fy);
      const int64_t o = (int64_t)(y0 + j - 2) * d.nx + x;
      rho_o[o] = rc;
      vx_o[o] = double(jxc / R(rc)) + Fx / (2.0 * rc);
      vy_o[o] = double(jyc / R(rc)) + Fy / (2.0 * rc);
      p_o[o] = pressure_of(rc, d);
    }
    rc = r;
    jxc = jx;
    jyc = jy;
#pragma unroll
    for (int a = 0; a < 9; ++a) f[a] = g[a];
  }
}

// Flat interface with normal x: mean density of each column (fixed order in y).
__global__ void k_colmean(const double* __restrict__ rho, int nx, int ny, double* __restrict__ out) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= nx) return;
  double s = 0.0;
  for (int y = 0; y < ny; ++y) s += rho[(int64_t)y * nx + x];
  out[x] = s / ny;
}

// Normal pressure across the profile (Eq. 25 with alpha = 0, beta = 3, plus the
// improved scheme's 2 G^2 sigma psi'^2 of Eq. 35); psi' and psi'' are central
// differences, periodic in x.
__global__ void k_normal_pressure(const double* __restrict__ rbar, RunDev d, double sigma,
                                  double* __restrict__ pn) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= d.nx) return;
  const int xm = x == 0 ? d.nx - 1 : x - 1, xp = x == d.nx - 1 ? 0 : x + 1;
  const double pm = sqrt(psi2_of(rbar[xm], d)), pc = sqrt(psi2_of(rbar[x], d)),
               pp = sqrt(psi2_of(rbar[xp], d));
  const double d1 = 0.5 * (pp - pm), d2 = (pp - 2.0 * pc) + pm;
  const double G = -d.mG;
  pn[x] = rbar[x] * (1.0 / 3.0) + 0.5 * G * pc * pc + (G / 12.0) * (3.0 * pc * d2) +
          2.0 * G * G * sigma * d1 * d1;
}

// Surface tension of one interface of a periodic flat slab with normal x, from
// the column-mean profile: gamma = (kappa + 2 G^2 sigma) sum_x psi'(x)^2 / 2,
// psi' central differences of psi(rbar) (Eq. 8), kappa = -G/6 (the
// P_b I + kappa grad psi grad psi form of the pressure tensor that Eq. (35)
// modifies, with kappa fixed by the second-order expansion of Eq. 3).  One
// block of 256 threads, fixed summation order.
__global__ __launch_bounds__(256) void k_surface_tension(const double* __restrict__ rbar, RunDev d,
                                                         double sigma, double* __restrict__ out) {
  __shared__ double sm[256];
  double acc = 0.0;
  for (int x = threadIdx.x; x < d.nx; x += 256) {
    const int xm = x == 0 ? d.nx - 1 : x - 1, xp = x == d.nx - 1 ? 0 : x + 1;
    const double d1 = 0.5 * (sqrt(psi2_of(rbar[xp], d)) - sqrt(psi2_of(rbar[xm], d)));
    acc += d1 * d1;
  }
  sm[threadIdx.x] = acc;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sm[threadIdx.x] += sm[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double G = -d.mG;
    out[0] = (-G / 6.0 + 2.0 * G * G * sigma) * sm[0] * 0.5;
  }
}

// Decode one stored population to FP64 exactly as the host decoder does:
// f = s + (w * rho_ref), two separately rounded operations.
__device__ __forceinline__ double decode(double v, int, double) { return v; }
__device__ __forceinline__ double decode(float v, int a, double rref) {
#pragma clang fp contract(off)
  const double wr = kW[a] * rref;
  return double(v) + wr;
}
__device__ __forceinline__ double decode(__half v, int a, double rref) {
#pragma clang fp contract(off)
  const double wr = kW[a] * rref;
  return double(__half2float(v)) + wr;
}

// Mass: per block, sum of round-to-nearest-even(rho * 2^40) (exact, 128-bit)
// and the FP64 sum; rho = sum_a f_a in direction order of the decoded
// populations.  Units of 64 columns of one row, dealt to the waves in turn (one
// division per unit, against one per node before: 67 -> 48 us on 2048 x 2048 FP64, 6.3
// TB/s with part of the lattice in the Infinity Cache).
template <typename S>
__global__ __launch_bounds__(256) void k_mass(const typename Store<S>::E* __restrict__ src, RunDev d,
                                              __int128* part_i, double* part_d) {
  __shared__ __int128 si[256];
  __shared__ double sd[256];
  const unsigned nxc = (unsigned)(d.nx + 63) >> 6;
  const unsigned units = nxc * (unsigned)d.ny;  // at most 2^31 / 3 for nx, ny >= 3
  const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __int128 acc_i = 0;
  double acc_d = 0.0;
  for (unsigned u = blockIdx.x * 4 + wave; u < units; u += gridDim.x * 4) {
    const int y = (int)(u / nxc), x = (int)(u - (unsigned)y * nxc) * 64 + (threadIdx.x & 63);
    if (x >= d.nx) continue;
    const int xm = x == 0 ? d.nx - 1 : x - 1, xp = x == d.nx - 1 ? 0 : x + 1;
    const int ym = y == 0 ? d.ny - 1 : y - 1, yp = y == d.ny - 1 ? 0 : y + 1;
    const int64_t P = d.plane;
    const int64_t r0 = (int64_t)y * d.rs, rm = (int64_t)ym * d.rs, rp = (int64_t)yp * d.rs;
    const int64_t idx[9] = {r0 + x,          P + r0 + xm,     2 * P + rm + x,
                            3 * P + r0 + xp, 4 * P + rp + x,  5 * P + rm + xm,
                            6 * P + rm + xp, 7 * P + rp + xp, 8 * P + rp + xm};
    double r = 0.0;
#pragma unroll
    for (int a = 0; a < 9; ++a)
      if (index_ok(idx[a], d.elems)) r += decode(src[idx[a]], a, d.rho_ref);
    acc_i += __double2ll_rn(r * 1099511627776.0);  // 2^40, exact scaling
    acc_d += r;
  }
  si[threadIdx.x] = acc_i;
  sd[threadIdx.x] = acc_d;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      si[threadIdx.x] += si[threadIdx.x + s];
      sd[threadIdx.x] += sd[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part_i[blockIdx.x] = si[0];
    part_d[blockIdx.x] = sd[0];
  }
}

// Final mass sums over the block partials (one block, fixed order: partials t, t +
// 256, ... per thread, then a tree):
// out[0], out[1] = low and high 64-bit words of the 128-bit integer sum, out[2]
// = the bits of the FP64 sum, out[3] = *flag (the first diverged step) where given.
// 2.7 us for 1024 partials, against 108 us by one thread.
__global__ __launch_bounds__(256) void k_mass_final(const __int128* __restrict__ part_i,
                                                    const double* __restrict__ part_d, int nblocks,
                                                    const unsigned long long* __restrict__ flag,
                                                    unsigned long long* __restrict__ out) {
  __shared__ __int128 si[256];
  __shared__ double sd[256];
  __int128 acc = 0;
  double m = 0.0;
  for (int i = threadIdx.x; i < nblocks; i += 256) {
    acc += part_i[i];
    m += part_d[i];
  }
  si[threadIdx.x] = acc;
  sd[threadIdx.x] = m;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      si[threadIdx.x] += si[threadIdx.x + s];
      sd[threadIdx.x] += sd[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = (unsigned long long)si[0];
    out[1] = (unsigned long long)(si[0] >> 64);
    out[2] = __double_as_longlong(sd[0]);
    out[3] = flag ? *flag : 0ull;
  }
}

}  // namespace lbm
