// Zone update: Flux-CT, flux divergence, geometric source, 1D_W inversion and
// bounds, fused in one kernel per substep; the fixup of failed zones; and the
// pointwise prim->cons / cons->prim calls.
//
//   U* = U(P_base) + dt (-sum_d [F_d(+) - F_d(-)]/dx_d + S(P_s)),
//   S_n = sqrt(-g) T^km d_n g_km / 2                                   (momenta)
//   P_out = invert(U*; guess P_s), then the bounds, then the fixup.
//
// Flux-CT (Implementation Notes, after Toth 2000): the B fluxes through each
// face are replaced by the mean of the two edge EMFs bounding it, each EMF
// being the mean of the four face fluxes around its edge; that keeps the
// corner divergence of sqrt(-g) B unchanged. On polar axes the axis EMFs and
// the hydrodynamic x2 fluxes through the axis are zero.
//
// 1D_W (Implementation Notes, after Noble et al. 2006): Newton on W' = W - D for
// the root of the energy equation, with v^2(W) and p(W) written so nothing
// cancels at small u/rho or small v; converged once |dW'| <= 1e-8 W, then two
// more steps; at most 50 steps; v^2 clamped to [0, 1 - 1e-12] while iterating
// (with the clamp's zero derivative). Failure: no convergence, W <= 0,
// v^2 >= 1 - 1e-12 or non-finite; a failed zone keeps the guess's hydro
// primitives and is flagged for the fixup.
//
// Bounds (Implementation Notes): Gamma <= gamma_max by rescaling u~; then
// rho >= max(rho_fl k, b^2/sigma_max); u >= max(u_fl k^gamma, beta_min b^2/(2(gamma-1)));
// rho >= u/uorho_max; k = 1/(r^2 (1 + r/10)).
#include <algorithm>
#include <type_traits>

#include "cks_geometry.h"
#include "kernels.h"

namespace {

constexpr int POINT_TX = 64, POINT_TY = 1;  // tile of the pointwise kernels
constexpr double INV_TOL = 1e-8;
constexpr int INV_EXTRA = 2;
constexpr int INV_MAXIT = 50;
constexpr double V2MAX = 1.0 - 1e-12;

// guess_l2: Gamma^2 of the guess. Divisions and square roots by rcp_full and
// rsqrt_full (an IEEE division is some ten instructions, and an iteration had
// three and a square root).
template <bool AXI>
__device__ bool invert_1dw(const double* U, const double* guess, double guess_l2, const ZoneGeo& g,
                           const UpdateParams& up, double* P) {
  const double a = g.alpha;
  const double ut0 = U[0] * g.igdet, ut1 = U[1] * g.igdet;
  const double q1 = U[2] * g.igdet, q2 = U[3] * g.igdet, q3 = U[4] * g.igdet;
  const double Bu1 = U[5] * g.igdet, Bu2 = U[6] * g.igdet, Bu3 = U[7] * g.igdet;
  const double D = a * ut0;
  const double Q1 = a * q1, Q2 = a * q2, Q3 = a * q3;
  const double B1 = a * Bu1, B2 = a * Bu2, B3 = a * Bu3;
  double bq = g.b1 * q1 + g.b2 * q2;
  if constexpr (!AXI) bq = bq + g.b3 * q3;
  const double qn_d = ut1 + (a - 1.0) * ut0 - bq;
  const double qt1 = g.h11 * Q1 + g.h12 * Q2 + g.h13 * Q3;
  const double qt2 = g.h12 * Q1 + g.h22 * Q2 + g.h23 * Q3;
  const double qt3 = g.h13 * Q1 + g.h23 * Q2 + g.h33 * Q3;
  const double qtsq = Q1 * qt1 + Q2 * qt2 + Q3 * qt3;
  const double qdb = Q1 * B1 + Q2 * B2 + Q3 * B3;
  const double qdb2 = qdb * qdb;
  double bl1, bl2, bl3;
  lower3<AXI>(g, B1, B2, B3, bl1, bl2, bl3);
  const double bsq = B1 * bl1 + B2 * bl2 + B3 * bl3;
  const double gf = up.gf;

  double x = (guess[0] + up.gam * guess[1]) * guess_l2 - D;
  int extra = -1;
  for (int it = 0; it < INV_MAXIT && extra < INV_EXTRA; ++it) {
    const double W = x + D;
    const double W2 = W * W, bw = bsq + W, Wbw = W * bw;
    const double rwb = rcp_full(Wbw);  // 1/(W bw), and 1/W = bw rwb
    const double iW = bw * rwb, iW2 = iW * iW, rwb2 = rwb * rwb;
    const double v2raw = (qtsq * W2 + qdb2 * (bw + W)) * rwb2;
    const double v2 = fmin(fmax(v2raw, 0.0), V2MAX);
    const double g2 = 1.0 - v2;
    const double is = rsqrt_full(g2), s = g2 * is;
    const double Ds = D * s;
    const double wmr = x * g2 - Ds * v2 * rcp_full(1.0 + s);
    const double f = qn_d + x - gf * wmr + 0.5 * bsq * (1.0 + v2) - 0.5 * qdb2 * iW2;
    double dv2 = -2.0 * (qtsq * (W2 * W) + qdb2 * (3.0 * Wbw + bsq * bsq)) * (rwb2 * rwb);
    if (v2raw > V2MAX || v2raw < 0.0) dv2 = 0.0;
    const double dp = gf * (g2 + (0.5 * D * is - W) * dv2);
    const double df = 1.0 - dp + 0.5 * bsq * dv2 + qdb2 * (iW2 * iW);
    const double dx = -f * rcp_ends(df);  // a derivative of 0 gives -inf, which halves W below
    double xn = x + dx;
    if (xn + D <= 0.0) xn = 0.5 * W - D;
    x = xn;
    if (extra < 0) {
      if (fabs(dx) <= INV_TOL * fabs(x + D)) extra = 0;
    } else {
      ++extra;
    }
  }
  const double W = x + D;
  const double bw = bsq + W;
  const double rwb = rcp_full(W * bw);
  const double v2 = (qtsq * W * W + qdb2 * (bw + W)) * (rwb * rwb);
  bool failed = (extra < 0) || !(W > 0.0) || !(v2 < V2MAX) || !isfinite(v2) || !isfinite(W);
  const double v2c = fmin(fmax(v2, 0.0), V2MAX);
  const double g2 = 1.0 - v2c;
  const double lor = rsqrt_full(g2), s = sqrt_by(g2, lor);
  P[0] = D * s;
  P[1] = div_by(x * g2 - D * s * v2c * rcp_full(1.0 + s), up.gam, up.igam);
  const double fac = lor * (W * rwb), qw = qdb * (bw * rwb);
  P[2] = fac * (qt1 + qw * B1);
  P[3] = fac * (qt2 + qw * B2);
  P[4] = fac * (qt3 + qw * B3);
  P[5] = Bu1;
  P[6] = Bu2;
  P[7] = Bu3;
  for (int v = 0; v < 5; ++v) failed = failed || !isfinite(P[v]);
  if (failed)
    for (int v = 0; v < 5; ++v) P[v] = guess[v];
  return failed;
}

template <bool AXI>
__device__ void apply_floors(double* P, const ZoneGeo& g, double rfl, double ufl, const UpdateParams& up) {
  double u1, u2, u3, B1, B2, B3;
  lower3<AXI>(g, P[2], P[3], P[4], u1, u2, u3);
  double l2 = P[2] * u1 + P[3] * u2 + P[4] * u3 + 1.0;
  double bt = P[5] * u1 + P[6] * u2 + P[7] * u3;
  const double gm2 = up.gamma_max * up.gamma_max;
  if (l2 > gm2) {
    const double sc = sqrt((gm2 - 1.0) / (l2 - 1.0));
    P[2] *= sc;
    P[3] *= sc;
    P[4] *= sc;
    bt *= sc;
    l2 = gm2;
  }
  lower3<AXI>(g, P[5], P[6], P[7], B1, B2, B3);
  const double Bsq = P[5] * B1 + P[6] * B2 + P[7] * B3;
  // b^2 = (B^2 + (b^t)^2) / (u^t)^2
  const double bsq = (Bsq + bt * bt) * (g.alpha * g.alpha * rcp_full(l2));
  double rho = fmax(fmax(P[0], rfl), bsq * up.isigma);
  const double u = fmax(fmax(P[1], ufl), up.beta_fl * bsq);
  rho = fmax(rho, u * up.iuorho);
  P[0] = rho;
  P[1] = u;
}

// contravariant u and b
template <bool AXI>
__device__ inline void contravariant(const double* P, const ZoneState& s, const ZoneGeo& g, double* u, double* b) {
  const double li = s.lor * g.ialpha;  // u^i = u~^i - Gamma beta^i / alpha
  u[0] = s.ut;
  u[1] = P[2] - li * g.b1;
  u[2] = P[3] - li * g.b2;
  u[3] = AXI ? P[4] : P[4] - li * g.b3;
  b[0] = s.bt;
#pragma unroll
  for (int m = 1; m < 4; ++m) b[m] = (P[4 + m] + s.bt * u[m]) * s.iut;
}

// sqrt(-g) T^km d_n g_km / 2 for n = 1, 2 (the coefficients of the table) of
// state P, s, added to rhs
__device__ inline void source_axi(const double* P, const ZoneState& s, const ZoneGeo& g, double gam, const double* ct,
                                  const Dims& d, int off, double* rhs) {
  double u[4], b[4], M[9];
  contravariant<true>(P, s, g, u, b);
  const double wb = P[0] + gam * P[1] + s.bsq;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int k = AXI_KM[q][0], m = AXI_KM[q][1];
    M[q] = wb * (u[k] * u[m]) - b[k] * b[m];
  }
  M[8] = (gam - 1.0) * P[1] + 0.5 * s.bsq;
  // coefficients C_S1 .. C_S1 + 17 in pairs: nine of x1, then nine of x2
  static_assert(!(C_S1 & 1) && C_S2 == C_S1 + 9, "pairs of the source coefficients");
  double S[2] = {0.0, 0.0};
#pragma unroll
  for (int c = 0; c < 18; c += 2) {
    const double2 q = zone_pair(ct, d, off, C_S1 + c);
    S[c / 9] = S[c / 9] + M[c % 9] * q.x;
    S[(c + 1) / 9] = S[(c + 1) / 9] + M[(c + 1) % 9] * q.y;
  }
  rhs[2] = rhs[2] + S[0];
  rhs[3] = rhs[3] + S[1];
}

// The same in Cartesian Kerr-Schild (sqrt(-g) = 1), with the centred
// differences of g_km taken here: six evaluations of the metric, some 600
// operations, against 33 coefficients read per zone (1.3 GB a launch on a
// 168^3 box, where the update took 0.61 ms reading them and takes 0.36).
__device__ inline void source_cks(const double* P, const ZoneState& s, const ZoneGeo& g, double gam, const CksBox& box,
                                  int i, int j, int k, double* rhs) {
  double u[4], b[4], T[10];
  contravariant<false>(P, s, g, u, b);
  const double wb = P[0] + gam * P[1] + s.bsq, pt = (gam - 1.0) * P[1] + 0.5 * s.bsq;
  const double ia2 = g.ialpha * g.ialpha, bi[3] = {g.b1, g.b2, g.b3};
  const double h[6] = {g.h11, g.h12, g.h13, g.h22, g.h23, g.h33};
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = m; n < 4; ++n) {
      // T^mn with g^-1 from gamma^ij, beta^i and alpha, times the multiplicity in the sum / 4 FD_DELTA
      const double gi = m == 0 ? (n == 0 ? -ia2 : bi[n - 1] * ia2)
                               : h[sidx(m, n) - 4] - bi[m - 1] * (bi[n - 1] * ia2);
      T[sidx(m, n)] = (wb * (u[m] * u[n]) - b[m] * b[n] + pt * gi) * ((m == n ? 0.25 : 0.5) / FD_DELTA);
    }
  double x[3];
  cks_centre(box, i, j, k, x);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    double gp[10], gm[10];
    const double e[3] = {c == 0 ? FD_DELTA : 0.0, c == 1 ? FD_DELTA : 0.0, c == 2 ? FD_DELTA : 0.0};
    cks_gcov(x[0] + e[0], x[1] + e[1], x[2] + e[2], box.a, gp);
    cks_gcov(x[0] - e[0], x[1] - e[1], x[2] - e[2], box.a, gm);
    double S = 0.0;
#pragma unroll
    for (int q = 0; q < 10; ++q) S = S + T[q] * (gp[q] - gm[q]);
    rhs[2 + c] = rhs[2 + c] + S;
    __builtin_amdgcn_sched_barrier(0);  // one direction at a time
  }
}

// b: block index within this job's grid (the update tile d.utx x d.uty, XCD-aware order)
// Z: where the zone's geometry comes from. SAME: the base state is the flux
// state (the predictor); its four-vectors then serve the conserved variables
// too (2 % of the predictor; in Cartesian Kerr-Schild keeping them across the
// source spills)
template <typename TF, int Z, bool SAME>
__device__ void update_body(const Dims& d, const double* __restrict__ cent, const UpdateParams& up,
                            const FluxOut<TF>& F, const double* Pb, const double* __restrict__ Ps, double* Pout,
                            int8_t* __restrict__ flags, double dt, Counters* ctr, int b) {
  constexpr bool AXI = Z == ZONE_AXI;
  const TileK tk = xcd_tile_k(b, d.utx, d.uty, d.n1, d.n3);
  const int i = tk.i0 + threadIdx.x;
  const int j = tk.j0 + threadIdx.y;
  const int k = tk.k;
  int failed = 0;
  if (tk.valid && i < d.n1 && j < d.n2) {
    const int c = cell_of(d, k, j, i);
    const size_t sv = (size_t)d.sv;
    const int s2 = d.s2, s3 = d.s3;
    const int off = tab_of(d, j, i);
    const double* ct = pair_plane(cent, d, k);
    double rhs[NV];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const TF* f = F.f3 + v * sv;
      rhs[v] = fma(-((double)buf_at(f + s3, c) - (double)buf_at(f, c)), up.idx3, buf_at(F.D + v * sv, c));
    }
    // Flux-CT: the zone's twelve edge EMFs (times four; in the flux precision)
    {
      const TF *E1 = F.e, *E2 = F.e + sv, *E3 = F.e + 2 * sv, *b2 = F.b, *b1 = F.b + sv;
      const TF e3_00 = buf_at(E3, c), e3_10 = buf_at(E3 + 1, c), e3_01 = buf_at(E3 + s2, c), e3_11 = buf_at(E3 + s2 + 1, c);
      const TF e1_00 = buf_at(E1, c) + buf_at(b2 - s3, c), e1_10 = buf_at(E1 + s2, c) + buf_at(b2 + s2 - s3, c);
      const TF e1_01 = buf_at(E1 + s3, c) + buf_at(b2, c), e1_11 = buf_at(E1 + s2 + s3, c) + buf_at(b2 + s2, c);
      const TF e2_00 = buf_at(E2, c) - buf_at(b1 - s3, c), e2_10 = buf_at(E2 + 1, c) - buf_at(b1 + 1 - s3, c);
      const TF e2_01 = buf_at(E2 + s3, c) - buf_at(b1, c), e2_11 = buf_at(E2 + s3 + 1, c) - buf_at(b1 + 1, c);
      // the face's field flux is half the sum of the two EMFs bounding it
      const TF h = TF(0.125);
      const double f1b2m = (double)(h * (e3_00 + e3_01)), f1b2p = (double)(h * (e3_10 + e3_11));
      const double f1b3m = (double)(-h * (e2_00 + e2_01)), f1b3p = (double)(-h * (e2_10 + e2_11));
      const double f2b1m = (double)(-h * (e3_00 + e3_10)), f2b1p = (double)(-h * (e3_01 + e3_11));
      const double f2b3m = (double)(h * (e1_00 + e1_01)), f2b3p = (double)(h * (e1_10 + e1_11));
      const double f3b1m = (double)(h * (e2_00 + e2_10)), f3b1p = (double)(h * (e2_01 + e2_11));
      const double f3b2m = (double)(-h * (e1_00 + e1_10)), f3b2p = (double)(-h * (e1_01 + e1_11));
      rhs[5] = -((f2b1p - f2b1m) * up.idx2 + (f3b1p - f3b1m) * up.idx3);
      rhs[6] = -((f1b2p - f1b2m) * up.idx1 + (f3b2p - f3b2m) * up.idx3);
      rhs[7] = -((f1b3p - f1b3m) * up.idx1 + (f2b3p - f2b3m) * up.idx2);
    }
    ZoneGeo g;
    zone_geo<Z>(g, ct, d, off, i, j, k);
    double ps[NV], U[NV], l2;
#pragma unroll
    for (int v = 0; v < NV; ++v) ps[v] = buf_at(Ps + v * sv, c);
    {
      ZoneState s;
      zone_state<AXI>(ps, g, s);
      l2 = s.l2;
      if constexpr (AXI) source_axi(ps, s, g, up.gam, ct, d, off, rhs);
      else source_cks(ps, s, g, up.gam, d.box, i, j, k, rhs);
      if constexpr (SAME) conserved<AXI>(ps, s, g, up.gam, U);
    }
    if constexpr (!SAME) {
      double pb[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) pb[v] = buf_at(Pb + v * sv, c);
      ZoneState s;
      zone_state<AXI>(pb, g, s);
      conserved<AXI>(pb, s, g, up.gam, U);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) U[v] = U[v] + dt * rhs[v];
    double pn[NV];
    failed = invert_1dw<AXI>(U, ps, l2, g, up, pn) ? 1 : 0;
    if (up.floors) {
      double rfl, ufl;
      zone_floors<Z>(rfl, ufl, ct, d, off);
      apply_floors<AXI>(pn, g, rfl, ufl, up);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) Pout[v * sv + c] = pn[v];
    flags[c] = (int8_t)failed;
    // Non-finite values left in the state. The hydro primitives of a zone
    // whose inversion succeeded are finite (a non-finite result is a failure,
    // and the bounds only take maxima with finite floors), and a failed zone's
    // are the fixup's to check: only the field can carry one out of here.
    if (!(isfinite(pn[5]) && isfinite(pn[6]) && isfinite(pn[7]))) atomicAdd(&ctr->bad, 1u);
  }
  block_count_to(failed, &ctr->fail, &ctr->fail_total);
}

// Bound by the address units (95 % busy: 71 loads a wave, 63 in the predictor,
// whose base state is the flux state) and HBM: 0.382 ms, predictor 0.341, on the
// 288 x 128 x 128 torus, 1.48 GB a launch of real traffic, 4.1 TB/s of the 4.9 a
// device copy reaches. With the 4 x 4 metric, its inverse and the 40 connection
// coefficients read per zone (66 values against 38 in pairs) and IEEE divisions
// both took 0.47 ms in the mean where they then took 0.35 (mixed precision 0.42
// against 0.29). (256, 3): at least three waves per SIMD. Held to
// four, the FP64 kernel takes 108 registers, keeps fewer loads in flight and
// 0.46 ms. Blocks that copy the tile's table to LDS and walk up 1 to 8 planes,
// carrying the x3 fluxes and EMFs between them, load 38 values instead of 71
// and take 0.42 ms: the copy, its barrier and each plane's loads wait one after
// the other.
template <typename TF, int Z, bool SAME>
__global__ __launch_bounds__(256, 3) void update_kernel(Dims d, const double* __restrict__ cent, UpdateParams up,
                                                        FluxOut<TF> F, const double* Pb, const double* __restrict__ Ps,
                                                        double* Pout, int8_t* __restrict__ flags, double dt,
                                                        const double* __restrict__ dt_dev, double dt_scale,
                                                        Counters* ctr) {
  if (dt_dev) dt = dt_scale * *dt_dev;
  update_body<TF, Z, SAME>(d, cent, up, F, Pb, Ps, Pout, flags, dt, ctr, (int)blockIdx.x);
}

// every job of a batch: predictor P -> P_h with dt/2, corrector (P, P_h) -> P with dt
template <typename TF, bool ALL_AXI, bool CORRECTOR>
__global__ __launch_bounds__(256, 3) void update_batch_kernel(BatchView bv) {
  const int* offs = bv.offs + PH_UPDATE * (bv.njobs + 1);
  const int jb = batch_job(offs, bv.njobs, (int)blockIdx.x);
  const JobDesc& J = bv.jobs[jb];
  const double dt = CORRECTOR ? *J.dt : 0.5 * *J.dt;
  const FluxOut<TF> F = flux_out<TF>(global_ptr((unsigned char*)J.F), J.d.sv);
  const double* Ps = global_ptr(CORRECTOR ? J.Ph : J.P);
  double* Pout = global_ptr(CORRECTOR ? J.P : J.Ph);
  const int b = (int)blockIdx.x - offs[jb];
  if (ALL_AXI || J.d.tk == 0)
    update_body<TF, ZONE_AXI, !CORRECTOR>(J.d, global_ptr(J.t.cent), J.up, F, global_ptr(J.P), Ps, Pout,
                                          global_ptr(J.flags), dt, global_ptr(J.ctr), b);
  else
    update_body<TF, ZONE_CKS, false>(J.d, global_ptr(J.t.cent), J.up, F, global_ptr(J.P), Ps, Pout, global_ptr(J.flags),
                                     dt, global_ptr(J.ctr), b);
}

// neighbour index along one direction for the fixup: across a periodic
// direction the zone on the other side of the seam, across a side whose ghost
// layer holds a neighbouring part's zones (halo bit) the ghost zone, else none
__device__ inline bool fixup_neighbour(int& x, int n, bool periodic, int halo, int lo_bit) {
  if (x >= 0 && x < n) return true;
  if (periodic) {
    x = x < 0 ? x + n : x - n;
    return true;
  }
  return (halo >> (lo_bit + (x < 0 ? 0 : 1))) & 1;
}

// failed zone <- mean of the hydro primitives of its non-failed neighbours
// among the 26 (values before any repair; across periodic directions and
// part boundaries as fixup_neighbour says), then the bounds
__device__ void fixup_body(const Dims& d, const double* __restrict__ cent, const UpdateParams& up, double* P,
                           const int8_t* __restrict__ flags, Counters* ctr, int halo, int b) {
  if (ctr->fail == 0u) return;
  const TileK tk = xcd_tile_k(b, d.utx, d.uty, d.n1, d.n3);
  const int i = tk.i0 + (int)threadIdx.x;
  const int j = tk.j0 + (int)threadIdx.y;
  const int k = tk.k;
  if (!tk.valid || i >= d.n1 || j >= d.n2) return;
  const int c = cell_of(d, k, j, i);
  if (!flags[c]) return;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  int cnt = 0;
  for (int dk = -1; dk <= 1; ++dk)
    for (int dj = -1; dj <= 1; ++dj)
      for (int di = -1; di <= 1; ++di) {
        if (dk == 0 && dj == 0 && di == 0) continue;
        int kk = k + dk, jj = j + dj, ii = i + di;
        if (!fixup_neighbour(ii, d.n1, up.periodic[0], halo, 0) ||
            !fixup_neighbour(jj, d.n2, up.periodic[1], halo, 2) ||
            !fixup_neighbour(kk, d.n3, up.periodic[2], halo, 4))
          continue;
        const int cc = cell_of(d, kk, jj, ii);
        if (flags[cc]) continue;
        for (int v = 0; v < 5; ++v) acc[v] += P[v * d.sv + cc];
        ++cnt;
      }
  double pn[NV];
  for (int v = 0; v < NV; ++v) pn[v] = P[v * d.sv + c];
  if (cnt > 0)
    for (int v = 0; v < 5; ++v) pn[v] = acc[v] / cnt;
  if (up.floors) {
    const int off = tab_of(d, j, i);
    const double* ct = pair_plane(cent, d, k);
    ZoneGeo g;
    zone_geo<ZONE_ANY>(g, ct, d, off, i, j, k);
    double rfl, ufl;
    zone_floors<ZONE_ANY>(rfl, ufl, ct, d, off);
    apply_floors<false>(pn, g, rfl, ufl, up);
  }
  bool fin = true;
  for (int v = 0; v < 5; ++v) {
    P[v * d.sv + c] = pn[v];
    fin = fin && isfinite(pn[v]);
  }
  if (!fin) atomicAdd(&ctr->bad, 1u);
}

// a grid of at most FIXUP_BLOCKS blocks strides over the tiles: when no zone
// failed (almost always) every block exits after one read of the counter
constexpr unsigned FIXUP_BLOCKS = 2048;  // a multiple of the XCD count
__global__ __launch_bounds__(256) void fixup_kernel(Dims d, const double* __restrict__ cent, UpdateParams up,
                                                    double* P, const int8_t* __restrict__ flags, Counters* ctr,
                                                    int halo, int ntiles) {
  if (ctr->fail == 0u) return;
  for (int b = (int)blockIdx.x; b < ntiles; b += (int)gridDim.x) fixup_body(d, cent, up, P, flags, ctr, halo, b);
}

// per blocks a job stride over its tiles, with the same early exit: a block per
// tile took 45 us a substep on 16 jobs of 10 million zones in all, none of them failed
__global__ __launch_bounds__(256) void fixup_batch_kernel(BatchView bv, int corrector, int per) {
  const int jb = (int)blockIdx.x / per;
  const JobDesc& J = bv.jobs[jb];
  Counters* ctr = global_ptr(J.ctr);
  if (ctr->fail == 0u) return;
  const int* offs = bv.offs + PH_UPDATE * (bv.njobs + 1);
  const int ntiles = offs[jb + 1] - offs[jb];
  for (int b = (int)blockIdx.x - jb * per; b < ntiles; b += per)
    fixup_body(J.d, global_ptr(J.t.cent), J.up, global_ptr(corrector ? J.P : J.Ph), global_ptr(J.flags), ctr, 0, b);
}

// prim->cons and cons->prim read and write 16 and 24 values a zone and are
// bound by that traffic; blocks in the update's XCD-aware order
template <int Z>
__global__ __launch_bounds__(256) void p2u_kernel(Dims d, const double* __restrict__ cent, double gam,
                                                  const double* __restrict__ P, double* __restrict__ U) {
  constexpr bool AXI = Z == ZONE_AXI;
  const TileK tk = xcd_tile_k((int)blockIdx.x, POINT_TX, POINT_TY, d.n1, d.n3);
  const int i = tk.i0 + (int)threadIdx.x, j = tk.j0 + (int)threadIdx.y, k = tk.k;
  if (!tk.valid || i >= d.n1 || j >= d.n2) return;
  const int c = cell_of(d, k, j, i);
  const size_t sv = (size_t)d.sv;
  double p[NV], u[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) p[v] = buf_at(P + v * sv, c);
  ZoneGeo g;
  zone_geo<Z>(g, pair_plane(cent, d, k), d, tab_of(d, j, i), i, j, k);
  ZoneState s;
  zone_state<AXI>(p, g, s);
  conserved<AXI>(p, s, g, gam, u);
#pragma unroll
  for (int v = 0; v < NV; ++v) U[v * sv + c] = u[v];
}

template <int Z>
__global__ __launch_bounds__(256) void u2p_kernel(Dims d, const double* __restrict__ cent, UpdateParams up,
                                                  const double* __restrict__ U, double* __restrict__ P,
                                                  int8_t* __restrict__ flags, Counters* ctr) {
  constexpr bool AXI = Z == ZONE_AXI;
  const TileK tk = xcd_tile_k((int)blockIdx.x, POINT_TX, POINT_TY, d.n1, d.n3);
  const int i = tk.i0 + (int)threadIdx.x, j = tk.j0 + (int)threadIdx.y, k = tk.k;
  int failed = 0;
  if (tk.valid && i < d.n1 && j < d.n2) {
    const int c = cell_of(d, k, j, i);
    const size_t sv = (size_t)d.sv;
    const int off = tab_of(d, j, i);
    const double* ct = pair_plane(cent, d, k);
    double u[NV], guess[NV], pn[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      u[v] = buf_at(U + v * sv, c);
      guess[v] = buf_at(P + v * sv, c);
    }
    ZoneGeo g;
    zone_geo<Z>(g, ct, d, off, i, j, k);
    double u1, u2, u3;
    lower3<AXI>(g, guess[2], guess[3], guess[4], u1, u2, u3);
    failed = invert_1dw<AXI>(u, guess, guess[2] * u1 + guess[3] * u2 + guess[4] * u3 + 1.0, g, up, pn) ? 1 : 0;
    if (up.floors) {
      double rfl, ufl;
      zone_floors<Z>(rfl, ufl, ct, d, off);
      apply_floors<AXI>(pn, g, rfl, ufl, up);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) P[v * sv + c] = pn[v];
    flags[c] = (int8_t)failed;
  }
  block_count_to(failed, &ctr->fail);
}

}  // namespace

namespace {

template <typename TF, bool SAME>
void update_for(const Dims& d, const Tables& t, const UpdateParams& up, const void* F, const double* Pb,
                const double* Ps, double* Pout, int8_t* flags, double dt, const double* dt_dev, double dt_scale,
                Counters* ctr, hipStream_t s) {
  const dim3 grd(xcd_grid(d.n1, d.n2, d.n3, d.utx, d.uty)), blk(d.utx, d.uty, 1);
  const FluxOut<TF> f = flux_out<TF>((unsigned char*)F, d.sv);
  if (d.tk != 0)
    hipLaunchKernelGGL((update_kernel<TF, ZONE_CKS, false>), grd, blk, 0, s, d, t.cent, up, f, Pb, Ps, Pout, flags, dt,
                       dt_dev, dt_scale, ctr);
  else
    hipLaunchKernelGGL((update_kernel<TF, ZONE_AXI, SAME>), grd, blk, 0, s, d, t.cent, up, f, Pb, Ps, Pout, flags, dt,
                       dt_dev, dt_scale, ctr);
}

template <typename TF>
void update_batch_for(const BatchView& bv, dim3 grd, bool corrector, hipStream_t s) {
  const dim3 blk(bv.utx, bv.uty, 1);
  if (bv.axi && corrector) hipLaunchKernelGGL((update_batch_kernel<TF, true, true>), grd, blk, 0, s, bv);
  else if (bv.axi) hipLaunchKernelGGL((update_batch_kernel<TF, true, false>), grd, blk, 0, s, bv);
  else if (corrector) hipLaunchKernelGGL((update_batch_kernel<TF, false, true>), grd, blk, 0, s, bv);
  else hipLaunchKernelGGL((update_batch_kernel<TF, false, false>), grd, blk, 0, s, bv);
}

}  // namespace

hipError_t launch_update(bool mixed, const Dims& d, const Tables& t, const UpdateParams& up, const void* F,
                         const double* Pb, const double* Ps, double* Pout, int8_t* flags, double dt,
                         const double* dt_dev, double dt_scale, Counters* ctr, hipStream_t s) {
  const auto launch = mixed ? (Pb == Ps ? update_for<float, true> : update_for<float, false>)
                            : (Pb == Ps ? update_for<double, true> : update_for<double, false>);
  launch(d, t, up, F, Pb, Ps, Pout, flags, dt, dt_dev, dt_scale, ctr, s);
  return hipGetLastError();
}

hipError_t launch_fixup(const Dims& d, const Tables& t, const UpdateParams& up, double* P, const int8_t* flags,
                        Counters* ctr, int halo, hipStream_t s) {
  const unsigned ntiles = xcd_grid(d.n1, d.n2, d.n3, d.utx, d.uty);
  const unsigned nblk = ntiles < FIXUP_BLOCKS ? ntiles : FIXUP_BLOCKS;
  hipLaunchKernelGGL(fixup_kernel, dim3(nblk), dim3(d.utx, d.uty, 1), 0, s, d, t.cent, up, P, flags, ctr, halo,
                     (int)ntiles);
  return hipGetLastError();
}

hipError_t launch_batch_update(const BatchView& bv, const int* totals, bool mixed, bool corrector, int which,
                               hipStream_t s) {
  const dim3 blk(bv.utx, bv.uty, 1), grd(totals[PH_UPDATE]);
  const int c = corrector ? 1 : 0;
  if (which & 1) {
    if (mixed) update_batch_for<float>(bv, grd, corrector, s);
    else update_batch_for<double>(bv, grd, corrector, s);
  }
  if (which & 2) {
    // as many blocks in all as a single job's fixup, 64 or more a job
    const int per = std::min(std::max(64, (int)FIXUP_BLOCKS / bv.njobs), totals[PH_UPDATE]);
    hipLaunchKernelGGL(fixup_batch_kernel, dim3(bv.njobs * per), blk, 0, s, bv, c, per);
  }
  return hipGetLastError();
}

hipError_t launch_prim_to_cons(const Dims& d, const Tables& t, double gam, const double* P, double* U,
                               hipStream_t s) {
  const dim3 blk(POINT_TX, POINT_TY, 1), grd(xcd_grid(d.n1, d.n2, d.n3, POINT_TX, POINT_TY));
  if (d.tk != 0) hipLaunchKernelGGL(p2u_kernel<ZONE_CKS>, grd, blk, 0, s, d, t.cent, gam, P, U);
  else hipLaunchKernelGGL(p2u_kernel<ZONE_AXI>, grd, blk, 0, s, d, t.cent, gam, P, U);
  return hipGetLastError();
}

hipError_t launch_cons_to_prim(const Dims& d, const Tables& t, const UpdateParams& up, const double* U,
                               double* P, int8_t* flags, Counters* ctr, hipStream_t s) {
  const dim3 blk(POINT_TX, POINT_TY, 1), grd(xcd_grid(d.n1, d.n2, d.n3, POINT_TX, POINT_TY));
  if (d.tk != 0) hipLaunchKernelGGL(u2p_kernel<ZONE_CKS>, grd, blk, 0, s, d, t.cent, up, U, P, flags, ctr);
  else hipLaunchKernelGGL(u2p_kernel<ZONE_AXI>, grd, blk, 0, s, d, t.cent, up, U, P, flags, ctr);
  return hipGetLastError();
}
