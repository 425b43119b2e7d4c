// Shared device definitions of the GRMHD zone-update library (gfx950).
//
// Layout (see grmhd.h): a state is [8][n3+6][n2+6][n1p] float64, x1 fastest.
// The results of the face-flux pass (FluxOut) use the same cells, a quantity
// of a lower face or edge at the cell it belongs to. Geometry tables hold the
// metric in 3+1 form, at the centres with the inverse of the spatial metric, the
// derivatives the source needs and the floor scales, and per direction at the
// faces. Axisymmetric coordinates store them as 2D tables [pair][n2+6][n1p][2]
// (k stride 0); Cartesian Kerr-Schild, whose metric depends on x3, has 3D tables
// [pair][n3+6][n2+6][n1p][2] (k stride = the state's), at the centres of the floor
// scales alone. The x3-face table of 2D tables holds centre values.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "grmhd.h"

// Multiply-adds are fused where one expression spells them out, and nowhere
// else: left to the back end ("fast", the default for HIP) the same function
// could round differently in two kernels, and a batch would not repeat a
// single context's bits.
#pragma clang fp contract(on)

#define NG GRMHD_NG
#define NV GRMHD_NVAR

// Centre table components, in pairs. MKS, FMKS and Minkowski (g_23 = beta^3 =
// 0): the 3+1 metric, the source coefficients S_k of x1 and x2 (eight
// derivatives each, then the pressure's), gamma^ij, 1/sqrt(-g), floor scales.
// Cartesian Kerr-Schild, whose metric and its differences the kernels evaluate
// themselves: floor scales and sqrt(-g).
// The source of the momentum along x^n is sqrt(-g) T^km d_n g_km / 2 (zero for
// the energy, the metric being stationary): the coefficients are sqrt(-g) d_n
// g_km, halved for k = m, and sqrt(-g) g^km d_n g_km / 2 for the pressure.
enum {
  C_G11 = 0, C_G12, C_G13, C_G22, C_G33, C_ALPHA, C_B1, C_B2, C_IALPHA, C_GDET,
  C_S1 = 10, C_S2 = 19, C_H11 = 28, C_H12, C_H13, C_H22, C_H23, C_H33, C_IGDET, C_RHOFL, C_UFL,
  K_RHOFL = 0, K_UFL, K_GDET,
  N_CENT = 64  // components the centre table has room for (38 or 3 are used; the allocation is part of the interface)
};
// the (k, m) of the eight derivatives of an axisymmetric table
constexpr int AXI_KM[8][2] = {{0, 0}, {0, 1}, {0, 3}, {1, 1}, {1, 2}, {1, 3}, {2, 2}, {3, 3}};

// face table components: the 3+1 form of the metric the face states are
// written in. g_ij is the spatial metric, beta^i = alpha^2 g^ti the shift,
// H = alpha^2 gamma^DD with gamma^ij the inverse of g_ij and D the face's
// direction. MKS, FMKS and Minkowski have g_23 = beta^3 = 0 identically
// (Kerr-Schild: g_theta phi = 0, g^t phi = 0), so their passes read the first
// F_AXI components only.
enum {
  F_G11 = 0, F_G12, F_G13, F_G22, F_G33, F_ALPHA,
  F_B1, F_B2, F_IALPHA, F_H, F_HGDET,  // 1/alpha, H, sqrt(-g)/2
  F_B3, F_AXI = F_B3 + 1, F_G23 = F_AXI, F_USED = F_G23 + 2,  // a pair is read at a time
  N_FACE = 22  // components a face table has room for (12 or 14 are used)
};

__host__ __device__ constexpr int sidx(int m, int n) {
  return (m <= n) ? (m * 4 - (m * (m - 1)) / 2 + (n - m)) : (n * 4 - (n * (n - 1)) / 2 + (m - n));
}

// Cartesian Kerr-Schild box
struct CksBox {
  double x0[3];  // x1min, x2min, x3min
  double dx[3];  // zone widths
  double a;
};

struct Dims {
  int n1, n2, n3;
  int p1, p2, p3;  // padded extents: n1p, n2 + 6, n3 + 6
  int s2;          // j stride (= p1)
  int s3;          // k stride (= p2 * p1)
  int sv;          // variable stride (= p3 * p2 * p1)
  int ts;          // table component stride (p2 * p1, or p3 * p2 * p1 for 3D tables)
  int tk;          // table k stride (0 for 2D tables, s3 for 3D)
  int stx, sty;    // thread-block tile (x1 x x2) asked for the sweeps
  int shape;       // and the block shape they use (sweep_shape)
  int sbx, sby;    // its extents
  int utx, uty;    // thread-block tile of the update and fixup
  int out_lo, out_hi;  // x1 lower / upper boundary is an outflow boundary
  CksBox box;          // Cartesian Kerr-Schild (tk != 0) only
};

__host__ __device__ inline int cell_of(const Dims& d, int k, int j, int i) {
  return (k + NG) * d.s3 + (j + NG) * d.s2 + (i + NG);
}
// point index of (j, i) within one x3 plane of the tables
__host__ __device__ inline int tab_of(const Dims& d, int j, int i) { return (j + NG) * d.s2 + (i + NG); }

// Loads through a buffer descriptor: a wave-uniform base pointer and one 32-bit
// byte offset a lane that every array of a kind shares (a component is < 4 GiB,
// checked at init). The pointer form costs a 64-bit vector add per load as soon
// as the compiler rewrites a family of addresses into a chain.
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xffffffffu, 0x00020000);
}
__device__ inline double buf_f64(const double* base, unsigned off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(buffer_of(base), (int)off, 0, 0));
}
__device__ inline double2 buf_pair(const double* base, unsigned off) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(buffer_of(base), (int)off, 0, 0));
}
__device__ inline float2 buf_pair(const float* base, unsigned off) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(buffer_of(base), (int)off, 0, 0));
}
__device__ inline float buf_f32(const float* base, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(buffer_of(base), (int)off, 0, 0));
}
// element off of an array
__device__ inline double buf_at(const double* base, int off) { return buf_f64(base, (unsigned)off * 8u); }
__device__ inline float buf_at(const float* base, int off) { return buf_f32(base, (unsigned)off * 4u); }

// The tables hold their components in pairs: component c of point off at
// (c & ~1) * ts + 2 * off + (c & 1), so one 16-byte (FP64) or 8-byte (FP32)
// load per lane brings two components. pair_plane gives the plane of x3 index
// k (the only plane of 2D tables).
__host__ __device__ inline size_t pair_index(int c, size_t ts, size_t off) {
  return (size_t)(c & ~1) * ts + 2 * off + (size_t)(c & 1);
}
template <typename S>
__host__ __device__ inline const S* pair_plane(const S* tab, const Dims& d, int k) {
  return tab + 2 * (size_t)(k + NG) * (size_t)d.tk;
}
template <typename S>
struct pair_of;
template <>
struct pair_of<double> {
  using type = double2;
};
template <>
struct pair_of<float> {
  using type = float2;
};

// geometry of one face
template <typename T>
struct FaceGeo {
  T g11, g12, g13, g22, g23, g33;  // g_ij
  T b1, b2, b3;                    // beta^i
  T alpha, ialpha, H, hgdet;
};

// from a face table (paired components; off as above, tab the plane from
// pair_plane); AXI: the coordinates have g_23 = beta^3 = 0
template <bool AXI, typename T, typename S>
__device__ inline void load_face_geo(FaceGeo<T>& g, const S* __restrict__ tab, int ts, int off) {
  using P2 = typename pair_of<S>::type;
  const unsigned bo = (unsigned)off * (unsigned)(2 * sizeof(S));
  auto ld = [&](int c0) -> P2 { return buf_pair(tab + (size_t)c0 * ts, bo); };
  const P2 a = ld(F_G11), b = ld(F_G13), c = ld(F_G33), d = ld(F_B1), e = ld(F_IALPHA), f = ld(F_HGDET);
  g.g11 = (T)a.x, g.g12 = (T)a.y;
  g.g13 = (T)b.x, g.g22 = (T)b.y;
  g.g33 = (T)c.x, g.alpha = (T)c.y;
  g.b1 = (T)d.x, g.b2 = (T)d.y;
  g.ialpha = (T)e.x, g.H = (T)e.y;
  g.hgdet = (T)f.x;
  g.b3 = T(0);
  g.g23 = T(0);
  if constexpr (!AXI) {
    g.b3 = (T)f.y;
    g.g23 = (T)ld(F_G23).x;
  }
}

// ---------------------------------------------------------------------------
// point physics (HARM variables; units GM = c = 1, b^2/2 magnetic pressure)

// 1/sqrt(x), 1/x and sqrt(x) to within about one unit in the last place,
// without the scaling and fix-up steps of the IEEE sequences: the hardware
// estimate r (FP64: 2^-24 or better) and one correction of third order in its
// residual e, r (1 + e/2 + 3/8 e^2) and r (1 + e + e^2). x must be a normal
// number away from the ends of the range.
__device__ inline double rsqrt_full(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * r), r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}
__device__ inline float rsqrt_full(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  return r * (1.5f - 0.5f * x * r * r);
}
__device__ inline double rcp_full(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ inline float rcp_full(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}
// and 1/0 = inf, 1/inf = 0, where the correction would make a NaN of them
__device__ inline double rcp_ends(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return e == e ? fma(r, fma(e, e, e), r) : r;
}
// A Goldschmidt step from the estimate, then one correction in the residual.
// x >= 0; 0 below the smallest argument the estimate is taken at
__device__ inline double sqrt_full(double x) {
  const double y = __builtin_amdgcn_rsq(fmax(x, 1e-290));
  const double g = x * y, h = 0.5 * y;
  const double e = fma(-g, h, 0.5);
  const double g1 = fma(g, e, g), h1 = fma(h, e, h);
  return fma(fma(-g1, g1, x), h1, g1);
}
// subnormal arguments count as 0: for numbers of order one, as side_speeds has them
__device__ inline float sqrt_full(float x) { return __builtin_amdgcn_sqrtf(x); }

// sqrt(x) from r = rsqrt_full(x) with one correction (x r alone is rounded twice:
// with it the inversion of a 24^3 box was 8.6e-17 from 80-bit arithmetic, with the
// correction and div_by 7.0e-17, as with IEEE roots and divisions)
__device__ inline double sqrt_by(double x, double r) {
  const double s = x * r;
  return fma(fma(-s, s, x), 0.5 * r, s);
}

// a / b from r = rcp_full(b) with one correction of the quotient, which rounds
// it as the IEEE division does but for rare last-place misses
__device__ inline double div_by(double a, double b, double r) {
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// One side of a face of direction D (1..3), in two steps: side_speeds finds the
// fast-magnetosonic speeds and what it needs for them, and once both sides'
// speeds have given ctop, side_flux adds the side's share of the
// local Lax-Friedrichs flux.
//
// Written in the 3+1 form, which needs the spatial metric, shift and lapse
// only and no index gymnastics with the four-metric:
//   u_i = g_ij u~^j, Gamma^2 = 1 + u~^i u_i, u^t = Gamma/alpha, 1/u^t = alpha/Gamma,
//   u_t = beta^i u_i - alpha Gamma, v^i = u^i/u^t = u~^i/u^t - beta^i,
//   B_mu = g_mu i B^i, B_t = beta^i B_i, b^t = B^i u_i,
//   b^i = B^i/u^t + b^t v^i, b_mu = (B_mu + b^t u_mu)/u^t, b^2 = (B^2 + (b^t)^2)/(u^t)^2.
// Speeds: c^2 = num/den with num = b^2 + gamma p, den = b^2 + w (v_A^2 +
// c_s^2 (1 - v_A^2) as one quotient). With m = den - num = rho + gamma (2 -
// gamma) u, q = num/Gamma^2 and y = u~^D/u^t the two roots of the dispersion
// relation are
//   z +- sqrt(q/(m + q) (H - z y)) - beta^D,  z = m y/(m + q),
// with no cancelling products, and quotients of densities alone: the product of
// two, q ((m + q) H - m y^2) under the root, is subnormal in FP32 where rho u is
// below 1e-38 (rho of 1e-14 and u of 3e-20 in a torus' outer atmosphere, with H
// = 1/r^2), and the hardware's root takes a subnormal number as 0.
// Flux and conserved variables differ in one factor only, v^D against 1 and
// b^D against b^t, so F + s U (s = ctop on the left, -ctop on the right) is the
// flux with the velocity W = v^D + s in place of v^D:
//   mass rho u^t W, field B^i W - B^D v^i,
//   T_mu = A u_mu - C B_mu, C = (B^D/u^t + b^t W)/u^t, A = (w + b^2) u^t W - C b^t,
// plus the pressure: p_tot in the momentum along D, s p_tot in the energy.
template <typename T>
struct FaceSide {
  T P[NV];
  T lor, iut, bt, bsq;  // Gamma, 1/u^t, b^t, b^2
  T cp, cm;             // speeds
};

// u_i = g_ij u~^j (or B_i)
template <bool AXI, typename G, typename T>
__device__ inline void lower3(const G& g, T v1, T v2, T v3, T& l1, T& l2, T& l3) {
  l1 = g.g11 * v1 + g.g12 * v2 + g.g13 * v3;
  l2 = g.g12 * v1 + g.g22 * v2;
  l3 = g.g13 * v1 + g.g33 * v3;
  if constexpr (!AXI) {
    l2 = l2 + g.g23 * v3;
    l3 = l3 + g.g23 * v2;
  }
}

template <int D, bool AXI, typename T>
__device__ inline void side_speeds(FaceSide<T>& s, const FaceGeo<T>& g, T gam) {
  const T* P = s.P;
  T u1, u2, u3, B1, B2, B3;
  lower3<AXI>(g, P[2], P[3], P[4], u1, u2, u3);
  const T l2 = P[2] * u1 + P[3] * u2 + P[4] * u3 + T(1);
  s.bt = P[5] * u1 + P[6] * u2 + P[7] * u3;
  lower3<AXI>(g, P[5], P[6], P[7], B1, B2, B3);
  const T Bsq = P[5] * B1 + P[6] * B2 + P[7] * B3;
  const T rl = rsqrt_full(l2);
  s.lor = l2 * rl;
  s.iut = g.alpha * rl;
  s.bsq = (Bsq + s.bt * s.bt) * (s.iut * s.iut);
  const T gp = gam * (gam - T(1));
  const T m = P[0] + (gam - gp) * P[1];
  const T q = (gp * P[1] + s.bsq) * (rl * rl);
  const T iA = rcp_full(m + q);
  const T y = P[1 + D] * s.iut;
  T mid = m * y * iA;
  const T r = sqrt_full(fmax((q * iA) * (g.H - mid * y), T(0)));
  if constexpr (D == 1) mid = mid - g.b1;
  else if constexpr (D == 2) mid = mid - g.b2;
  else if constexpr (!AXI) mid = mid - g.b3;
  s.cp = mid + r;
  s.cm = mid - r;
}

// f: mass, energy, 3 momenta, then the two transverse field components
// (ascending), divided by sqrt(-g)
template <int D, bool AXI, typename T>
__device__ inline void side_flux(const FaceSide<T>& s, const FaceGeo<T>& g, T gam, T st, T* f) {
  const T* P = s.P;
  T u1, u2, u3, B1, B2, B3;
  lower3<AXI>(g, P[2], P[3], P[4], u1, u2, u3);
  lower3<AXI>(g, P[5], P[6], P[7], B1, B2, B3);
  T ult = g.b1 * u1 + g.b2 * u2 - g.alpha * s.lor;
  T Blt = g.b1 * B1 + g.b2 * B2;
  T W = P[1 + D] * s.iut + st;
  if constexpr (D == 1) W = W - g.b1;
  else if constexpr (D == 2) W = W - g.b2;
  if constexpr (!AXI) {
    ult = ult + g.b3 * u3;
    Blt = Blt + g.b3 * B3;
    if constexpr (D == 3) W = W - g.b3;
  }
  const T BD = P[4 + D];
  const T m = s.lor * g.ialpha * W;
  const T C = (BD * s.iut + s.bt * W) * s.iut;
  const T A = (P[0] + gam * P[1] + s.bsq) * m - C * s.bt;
  const T pt = (gam - T(1)) * P[1] + T(0.5) * s.bsq;
  f[0] = P[0] * m;
  f[1] = A * ult - C * Blt + st * pt + f[0];
  f[2] = A * u1 - C * B1;
  f[3] = A * u2 - C * B2;
  f[4] = A * u3 - C * B3;
  f[1 + D] = f[1 + D] + pt;
  constexpr int a = D == 1 ? 2 : 1, b = D == 3 ? 2 : 3;
  const T va = P[1 + a] * s.iut - (D == 1 ? g.b2 : g.b1);
  T vb = P[1 + b] * s.iut;
  if constexpr (D == 3) vb = vb - g.b2;
  else if constexpr (!AXI) vb = vb - g.b3;
  f[5] = P[4 + a] * W - BD * va;
  f[6] = P[4 + b] * W - BD * vb;
}

// Geometry of a zone centre in the same 3+1 form, with gamma^ij.
struct ZoneGeo {
  double g11, g12, g13, g22, g23, g33;
  double b1, b2, b3;
  double alpha, ialpha, gdet, igdet;
  double h11, h12, h13, h22, h23, h33;
};

// what the conserved variables and the source need of primitives P
struct ZoneState {
  double u1, u2, u3, B1, B2, B3;       // u_i, B_i
  double l2, lor, ut, iut, bt, bsq;    // Gamma^2, Gamma, u^t, 1/u^t, b^t, b^2
};

template <bool AXI>
__device__ inline void zone_state(const double* P, const ZoneGeo& g, ZoneState& s) {
  lower3<AXI>(g, P[2], P[3], P[4], s.u1, s.u2, s.u3);
  s.l2 = P[2] * s.u1 + P[3] * s.u2 + P[4] * s.u3 + 1.0;
  s.bt = P[5] * s.u1 + P[6] * s.u2 + P[7] * s.u3;
  lower3<AXI>(g, P[5], P[6], P[7], s.B1, s.B2, s.B3);
  const double Bsq = P[5] * s.B1 + P[6] * s.B2 + P[7] * s.B3;
  const double rl = rsqrt_full(s.l2);
  s.lor = sqrt_by(s.l2, rl);
  s.ut = s.lor * g.ialpha;
  s.iut = g.alpha * rl;
  s.bsq = (Bsq + s.bt * s.bt) * (s.iut * s.iut);
}

// sqrt(-g) (rho u^t, T^t_t + rho u^t, T^t_i, B^i)
template <bool AXI>
__device__ inline void conserved(const double* P, const ZoneState& s, const ZoneGeo& g, double gam, double* U) {
  const double rt = P[0] * s.ut;
  const double C = s.bt * s.iut;
  const double A = (P[0] + gam * P[1] + s.bsq) * s.ut - C * s.bt;
  const double pt = (gam - 1.0) * P[1] + 0.5 * s.bsq;
  double ut = g.b1 * s.u1 + g.b2 * s.u2 - g.alpha * s.lor, Bt = g.b1 * s.B1 + g.b2 * s.B2;
  if constexpr (!AXI) {
    ut = ut + g.b3 * s.u3;
    Bt = Bt + g.b3 * s.B3;
  }
  U[0] = g.gdet * rt;
  U[1] = g.gdet * (A * ut - C * Bt + pt + rt);
  U[2] = g.gdet * (A * s.u1 - C * s.B1);
  U[3] = g.gdet * (A * s.u2 - C * s.B2);
  U[4] = g.gdet * (A * s.u3 - C * s.B3);
  U[5] = g.gdet * P[5];
  U[6] = g.gdet * P[6];
  U[7] = g.gdet * P[7];
}

// ---------------------------------------------------------------------------
// reconstruction

// Half the monotonised-central slope of a zone from its left and right
// differences: min(|dm|, |dp|, |dm + dp|/4) with the sign of the flow, 0 at an
// extremum. The 0 or 1 of that test multiplies the slope (one select instead of
// two for a 64-bit zero).
template <typename T>
struct McSlope {
  T h, one;
  __device__ McSlope(T dm, T dp) {
    const T c = T(0.25) * (dm + dp);
    h = copysign(fmin(fmin(fabs(dm), fabs(dp)), fabs(c)), c);
    one = dm * dp > T(0) ? T(1) : T(0);
  }
  __device__ T above(T p) const { return fma(h, one, p); }
  __device__ T below(T p) const { return fma(-h, one, p); }
};

// Value at the right edge of the middle zone of (x1..x5), point-value WENO5
// with Jiang-Shu smoothness indicators b_k and linear weights (1/16, 5/8, 5/16):
// weights d_k / (eps + b_k)^2, normalised, eps = 1e-26. Written in the
// differences d_k = x_(k+1) - x_k: the candidates are x3 plus two of them, and
// 4 b_k = (13/3) t_k^2 + u_k^2 with t_k their differences. e_k = 4 (eps + b_k).
template <typename T>
struct Weno {
  T d1, d2, d3, d4, e0, e1, e2, m;
  __device__ Weno(T x1, T x2, T x3, T x4, T x5) {
    d1 = x2 - x1;
    d2 = x3 - x2;
    d3 = x4 - x3;
    d4 = x5 - x4;
    const T t0 = d2 - d1, t1 = d3 - d2, t2 = d4 - d3;
    const T u0 = T(2) * d2 + t0, u1 = d2 + d3, u2 = T(2) * d3 - t2;
    constexpr T C = T(13.0 / 3.0), EPS = T(4e-26);
    e0 = u0 * u0 + EPS;
    e1 = u1 * u1 + EPS;
    e2 = u2 * u2 + EPS;
    e0 = (C * t0) * t0 + e0;
    e1 = (C * t1) * t1 + e1;
    e2 = (C * t2) * t2 + e2;
    m = fmin(fmin(e0, e1), e2);
  }
  // x3 and the mean of the candidates' distances from it with weights a_k
  __device__ T mean(T x3, T a0, T a1, T a2) const {
    const T q0 = T(0.875) * d2 - T(0.375) * d1;
    const T q1 = T(0.375) * d3 + T(0.125) * d2;
    const T q2 = T(0.625) * d3 - T(0.125) * d4;
    return (a0 * q0 + a1 * q1 + a2 * q2) * rcp_full(a0 + a1 + a2) + x3;
  }
  // the same at the left edge: what mean gives with the zones in reverse order
  // (d_k <-> -d_(5-k), a_0 <-> a_2), bit for bit
  __device__ T mirrored(T x3, T a0, T a1, T a2) const {
    const T q0 = T(0.375) * d4 - T(0.875) * d3;
    const T q1 = T(-0.375) * d2 - T(0.125) * d3;
    const T q2 = T(0.125) * d1 - T(0.625) * d2;
    return (a2 * q0 + a1 * q1 + a0 * q2) * rcp_full(a2 + a1 + a0) + x3;
  }
};

// Over a common denominator, scaled by the smallest e_k so nothing leaves the
// double range: with r_k = e_k / e_min >= 1 the weights are proportional to d_k
// times the product of the other two r_j^2 (two reciprocals instead of four).
__device__ inline double weno5_edge(double x1, double x2, double x3, double x4, double x5) {
  const Weno<double> w(x1, x2, x3, x4, x5);
  const double im = rcp_full(w.m);
  // r_k <= 1e60 keeps the products of two squares finite; such a weight is 0 anyway
  const double r0 = fmin(w.e0 * im, 1e60), r1 = fmin(w.e1 * im, 1e60), r2 = fmin(w.e2 * im, 1e60);
  const double s0 = r0 * r0, s1 = r1 * r1, s2 = r2 * r2;
  return w.mean(x3, s1 * s2, 10.0 * (s0 * s2), 5.0 * (s0 * s1));
}
// both edges of the middle zone, which share the smoothness indicators
__device__ inline void weno5_edges(double x1, double x2, double x3, double x4, double x5, double& left, double& right) {
  const Weno<double> w(x1, x2, x3, x4, x5);
  const double im = rcp_full(w.m);
  const double r0 = fmin(w.e0 * im, 1e60), r1 = fmin(w.e1 * im, 1e60), r2 = fmin(w.e2 * im, 1e60);
  const double s0 = r0 * r0, s1 = r1 * r1, s2 = r2 * r2;
  const double p0 = s1 * s2, p1 = 10.0 * (s0 * s2), p2 = s0 * s1;
  right = w.mean(x3, p0, p1, 5.0 * p2);
  left = w.mirrored(x3, 5.0 * p0, p1, p2);
}

// FP32 form: eps^2 = 1e-52 is below the float range, so the weights use the
// ratios r_k = e_min / e_k in (0, 1]: d_k r_k^2, normalised; the term of the
// smallest e_k has r = 1, so the sum is at least its d_k. Ratios by the
// hardware rcp (about 1 ulp), far below the float rounding of the inputs.
__device__ inline float weno5_edge(float x1, float x2, float x3, float x4, float x5) {
  const Weno<float> w(x1, x2, x3, x4, x5);
  const float r0 = w.m * __builtin_amdgcn_rcpf(w.e0), r1 = w.m * __builtin_amdgcn_rcpf(w.e1),
              r2 = w.m * __builtin_amdgcn_rcpf(w.e2);
  return w.mean(x3, r0 * r0, 10.0f * (r1 * r1), 5.0f * (r2 * r2));
}
__device__ inline void weno5_edges(float x1, float x2, float x3, float x4, float x5, float& left, float& right) {
  const Weno<float> w(x1, x2, x3, x4, x5);
  const float r0 = w.m * __builtin_amdgcn_rcpf(w.e0), r1 = w.m * __builtin_amdgcn_rcpf(w.e1),
              r2 = w.m * __builtin_amdgcn_rcpf(w.e2);
  const float p0 = r0 * r0, p1 = 10.0f * (r1 * r1), p2 = r2 * r2;
  right = w.mean(x3, p0, p1, 5.0f * p2);
  left = w.mirrored(x3, 5.0f * p0, p1, p2);
}

// ---------------------------------------------------------------------------
// XCD-aware block mapping
//
// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.
// Stencil kernels use a 1D grid of 8 * ntiles * chunk blocks, where a tile is
// a tx x ty (x1, x2) patch (one thread per cell, the block's shape) and
// chunk = ceil(nk / 8): XCD x receives, in order, every tile with k in
// [x*chunk, (x+1)*chunk). Consecutive blocks on one XCD then share the tile's
// 2D geometry and its neighbouring x3 planes in that XCD's L2 instead of
// refetching them once per x3 plane.

constexpr int NXCD = 8;
constexpr int TILE_X = 64;   // default tiles: face fluxes 64 x 8 (512 threads), update 64 x 1
constexpr int SWEEP_TILE_X = 64;
constexpr int SWEEP_TILE_Y = 8;
constexpr int TILE_Y = 1;
constexpr int SWEEP_MAX_THREADS = 512;   // launch bounds of the sweep kernels
constexpr int UPDATE_MAX_THREADS = 256;  // launch bounds of the update and fixup kernels

// What the face-flux pass leaves for the update, per cell:
//   D   minus the divergence of the five hydrodynamic fluxes in x1 and x2;
//   f3  the five hydrodynamic x3 fluxes;
//   e   four times the EMF of the cell's lower x1, x2 and x3 edge, the first
//       two without the flux of the plane below,
//   b   which are the x2 and the x1 flux of B3;
//   m   the mass fluxes through the lower x1 and x2 face (electron steps only;
//       the x3 one is f3's first).
// and the predictor's electron pass leaves
//   r   sqrt(-g) rho u^t of the base state for the corrector's.
// T is the precision of the fluxes. 18 values a cell, which fill 96 of the 96
// bytes there is room for with T = float (three flux arrays of a state's shape).
template <typename T>
struct FluxOut {
  double *D, *r;
  T *f3, *e, *b, *m;
};
template <typename T>
__host__ __device__ inline FluxOut<T> flux_out(unsigned char* base, int sv) {
  FluxOut<T> o;
  o.D = (double*)base;
  o.r = o.D + 5 * (size_t)sv;
  o.f3 = (T*)(o.r + sv);
  o.e = o.f3 + 5 * (size_t)sv;
  o.b = o.e + 3 * (size_t)sv;
  o.m = o.b + 2 * (size_t)sv;
  return o;
}

// Its tiles cover the cells -1..n. They overlap by two columns in x1 (a face needs
// the cell before it, a divergence the face after it) and one row in x2; the last
// tile's last column, which has no face after it, may be cell n, which has no
// divergence.
__host__ __device__ inline int sweep_tiles_x1(int n, int b) { return (n + b - 3) / (b - 2); }
__host__ __device__ inline int sweep_tiles_x2(int n, int b) { return (n + 1 + b - 2) / (b - 1); }
// Block shapes of the face-flux pass, bx x by threads in rows no longer than a
// wave: the large one is 64 x 8, or 32 x 16 for FP64 WENO5, whose 64 x 8 plane
// and exchange take 86 KB of LDS and leave one block a CU; the small one 32 x 8,
// the narrow one 16 x 8.
enum { SWEEP_LARGE = 0, SWEEP_SMALL, SWEEP_NARROW, SWEEP_SHAPES };
__host__ __device__ constexpr int sweep_bx(int shape, int recon, bool mixed) {
  return shape == SWEEP_NARROW ? 16 : shape == SWEEP_SMALL || (recon == GRMHD_RECON_WENO5 && !mixed) ? 32 : 64;
}
__host__ __device__ constexpr int sweep_by(int shape, int recon, bool mixed) {
  return shape == SWEEP_LARGE ? 512 / sweep_bx(shape, recon, mixed) : 8;
}
// blocks of a grid in the shape (bx, by)
inline long long sweep_grid(const Dims& d, int bx, int by) {
  return (long long)sweep_tiles_x1(d.n1, bx) * sweep_tiles_x2(d.n2, by) * ((d.n3 + 2 + NXCD - 1) / NXCD) * NXCD;
}
// blocks of a pass (over one grid, or the jobs of a batch) in each shape
struct SweepBlocks {
  long long n[SWEEP_SHAPES] = {0, 0, 0};
  void add(const Dims& d, int recon, bool mixed) {
    for (int q = 0; q < SWEEP_SHAPES; ++q) n[q] += sweep_grid(d, sweep_bx(q, recon, mixed), sweep_by(q, recon, mixed));
  }
};
// The shape of a pass. Tiles asked for (stx x sty other than the default) name
// it: 16 zones wide the narrow one, otherwise above 256 threads the large one.
// Left to the grid, the large shape, but
// * below 1024 of its blocks, two rounds of the two a CU holds, the small one:
//   the large would leave CUs idle (64 x 64 x 1: 13.7 us against 10.9);
// * the small one where it covers the grid with 7/8 of the threads or less
//   (30 x 200 x 100: 89 us against 52; 131 x 67 x 45, 5/6: 51 against 44; 192 x 96 x
//   64, 7/8: 139 against 127; with equal threads 160 x 96 x 48 takes 83 against 77, but
//   288 x 128 x 128 0.42 ms against 0.46, mixed 0.33 against 0.38);
// * the narrow one where it takes 2/3 of the threads or less, at n1 <= 14 (8 x 256
//   x 128: 70 us against 43; with equal threads, 24 x 128 x 128, 45 against 50; with
//   3/4, 40^3 mixed, 15.9 against 16.6), in FP64 WENO5, whose large shape spans 15
//   rows, 5/6 where it fills the device (62 x 7 x 900: 168 us against 152; 64^3 75
//   against 71; with fewer blocks, 64 x 64 x 1, 17.7 against 21.5).
inline int sweep_shape(int stx, int sty, const SweepBlocks& blocks, int recon, bool mixed) {
  if (stx != SWEEP_TILE_X || sty != SWEEP_TILE_Y)
    return stx < 32 ? SWEEP_NARROW : stx * sty > 256 ? SWEEP_LARGE : SWEEP_SMALL;
  const auto threads = [&](int q) { return blocks.n[q] * sweep_bx(q, recon, mixed) * sweep_by(q, recon, mixed); };
  int shape = SWEEP_LARGE;
  if (blocks.n[SWEEP_LARGE] < 1024 || 8 * threads(SWEEP_SMALL) <= 7 * threads(SWEEP_LARGE)) shape = SWEEP_SMALL;
  const bool rows = recon == GRMHD_RECON_WENO5 && !mixed && blocks.n[SWEEP_NARROW] >= 1024;
  if (6 * threads(SWEEP_NARROW) <= (rows ? 5 : 4) * threads(shape)) shape = SWEEP_NARROW;
  return shape;
}
inline void set_sweep_shape(Dims& d, int shape, int recon, bool mixed) {
  d.shape = shape;
  d.sbx = sweep_bx(shape, recon, mixed);
  d.sby = sweep_by(shape, recon, mixed);
}
struct SweepTile {
  int i0, j0, k;   // first cell of the tile and its plane
  bool valid;
};
// XCD x takes a slab of planes, tile by tile with x2 fastest: a tile's planes
// share its geometry and their x3 stencils in the XCD's L2, and the next tile
// finds the rows it shares with them there
__device__ inline SweepTile sweep_tile(const Dims& d, int bx, int by, int b) {
  const int ty = sweep_tiles_x2(d.n2, by), planes = d.n3 + 2, chunk = (planes + NXCD - 1) / NXCD;
  const int x = b % NXCD, w = b / NXCD, tile = w / chunk;
  SweepTile t;
  t.k = -1 + x * chunk + (w - tile * chunk);
  t.i0 = -1 + (tile / ty) * (bx - 2);
  t.j0 = -1 + (tile % ty) * (by - 1);
  t.valid = t.k <= d.n3;
  return t;
}

struct TileK {
  int i0, j0, k;
  bool valid;
};

// b: block index within this job's grid (a multiple-of-8 offset from the
// launch's block index, so b % 8 is still the XCD)
__device__ inline TileK xcd_tile_k(int b, int tx, int ty, int ni, int nk) {
  const int tiles_x = (ni + tx - 1) / tx;
  const int chunk = (nk + NXCD - 1) / NXCD;
  const int x = b % NXCD, w = b / NXCD;
  const int tile = w / chunk;
  TileK t;
  t.k = x * chunk + (w - tile * chunk);
  t.i0 = (tile % tiles_x) * tx;
  t.j0 = (tile / tiles_x) * ty;
  t.valid = t.k < nk;
  return t;
}

// 1D grid size for ni x nj x nk cells in tx x ty tiles
inline unsigned xcd_grid(int ni, int nj, int nk, int tx, int ty) {
  const int tiles = ((ni + tx - 1) / tx) * ((nj + ty - 1) / ty);
  const int chunk = (nk + NXCD - 1) / NXCD;
  return (unsigned)(NXCD * tiles * chunk);
}

// ---------------------------------------------------------------------------
// block reductions

__device__ inline double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ inline int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// max of a non-negative double over the block, then one atomic max on the
// IEEE bit pattern (order-preserving for non-negative values). Callers map NaN
// to +inf first so a non-finite speed survives the reduction.
__device__ inline void block_max_to(double v, unsigned long long* dst) {
  __shared__ double part[16];
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  v = wave_max(v + 0.0);
  if ((tid & 63) == 0) part[tid >> 6] = v;
  __syncthreads();
  if (tid == 0) {
    double m = part[0];
    for (int w = 1; w < (nthr + 63) / 64; ++w) m = fmax(m, part[w]);
    atomicMax(dst, (unsigned long long)__double_as_longlong(m + 0.0));
  }
}

// the maximum of non-negative values over a wave, in its last lane, by moves
// between lanes (a shuffle goes through LDS)
template <int CTRL>
__device__ inline double dpp_max(double v) {
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  return fmax(v, __hiloint2double(hi, lo));
}
__device__ inline double wave_max_last(double v) {
  v = dpp_max<0x111>(v);  // row_shr 1, 2, 4, 8: the last lane of each row of 16
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  v = dpp_max<0x118>(v);
  v = dpp_max<0x142>(v);  // row_bcast 15 and 31: across the rows
  return dpp_max<0x143>(v);
}

// block_max_to for three values at once into dst[0..2]: one barrier, and
// the atomic only where the block's maximum exceeds the running one (values
// only grow, so a stale read can only cost an unneeded atomic)
__device__ inline void block_max3_to(double a, double b, double c, unsigned long long* dst) {
  __shared__ double part3[3][16];
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  a = wave_max_last(a + 0.0);
  b = wave_max_last(b + 0.0);
  c = wave_max_last(c + 0.0);
  if ((tid & 63) == 63) {
    part3[0][tid >> 6] = a;
    part3[1][tid >> 6] = b;
    part3[2][tid >> 6] = c;
  }
  __syncthreads();
  if (tid < 3) {
    double m = part3[tid][0];
    for (int w = 1; w < (nthr + 63) / 64; ++w) m = fmax(m, part3[tid][w]);
    const unsigned long long bits = (unsigned long long)__double_as_longlong(m + 0.0);
    if (__hip_atomic_load(dst + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < bits) atomicMax(dst + tid, bits);
  }
}

// block sum of v, then one atomic add into dst (and into dst2 when given)
__device__ inline void block_count_to(int v, unsigned int* dst, unsigned int* dst2 = nullptr) {
  __shared__ int cpart[16];
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  v = wave_sum(v);
  if ((tid & 63) == 0) cpart[tid >> 6] = v;
  __syncthreads();
  if (tid == 0) {
    int s = 0;
    for (int w = 0; w < (nthr + 63) / 64; ++w) s += cpart[w];
    if (s) {
      atomicAdd(dst, (unsigned int)s);
      if (dst2) atomicAdd(dst2, (unsigned int)s);
    }
  }
}
