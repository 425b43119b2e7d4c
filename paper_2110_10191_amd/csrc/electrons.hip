// Electron heating (Implementation Notes: the dissipation is tracked and split
// between ions and electrons after Ressler et al. 2015, with the heating
// models of Kawazura et al. 2019, Werner et al. 2018, Rowan et al. 2017,
// Howes 2010 and Sharma et al. 2007). One pass per substep after the fluid
// update, bounds and fixup, for both entropies K (K_tot = P_gas / rho^gamma and
// K_e = P_e / rho^gamma_e, gamma_e = 4/3):
//
//   advection: U_K = sqrt(-g) rho_b u^t_b K_b - dt sum_d [F_K(+) - F_K(-)] / dx_d,
//     F_K = F_mass K*, K* the face value (the fluid's reconstruction) on the
//     upwind side of the mass flux; the mass flux through a polar axis is 0.
//     The predictor's pass leaves sqrt(-g) rho u^t of the base state for the
//     corrector's, whose update has overwritten it;
//
//   heating: u <= 3 rho^gamma / (gamma - 1) (P_gas / rho^gamma < 3); with D =
//   sqrt(-g) rho u^t of the new state, K_adv = U_K / D and K = (gamma - 1) u /
//   rho^gamma,
//     K_e = K_e,adv + f_e (gamma_e - 1)/(gamma - 1) rho^(gamma - gamma_e) (K - K_tot,adv)
//   (the electrons receive the fraction f_e of the dissipated internal
//   energy), bounded to [0, rho^(gamma - gamma_e) K] (0 <= P_e <= P_gas), and
//   K_tot = K.
//
// f_e is a constant or a model of beta_i = P_i / (b^2/2), T_e/T_i = P_e / P_i
// (P_i = P_gas - P_e), sigma = b^2/rho and sigma_w = b^2 / (rho + u + P_gas):
//   Kawazura: Q_i/Q_e = 35 / (1 + (beta_i/15)^-1.4 exp(-0.1 T_e/T_i));
//   Werner:   f_e = (1 + sqrt((sigma/5) / (2 + sigma/5))) / 4;
//   Rowan:    f_e = exp(-max(1 - beta_i/beta_max, 0)^3.3 / (1 + 1.2 sigma_w^0.7)) / 2,
//             beta_max = 1/(4 sigma_w);
//   Howes:    theta = T_i/T_e, Q_i/Q_e = 0.92 (c2^2 + beta_i^x)/(c3^2 + beta_i^x)
//             sqrt(theta m_p/m_e) exp(-1/beta_i), x = 2 - 0.2 log10 theta,
//             c2 = 1.6/theta, c3 = 18 + 5 log10 theta for theta > 1,
//             c2 = 1.2/theta, c3 = 18 otherwise, beta_i^x capped at e^700;
//   Sharma:   Q_e/Q_i = sqrt(T_e/T_i) / 3, i.e. Q_i/Q_e = 3 sqrt(T_i/T_e);
// with f_e = 1 / (1 + Q_i/Q_e) where a ratio is given.
#include "cks_geometry.h"
#include "kernels.h"

namespace {

constexpr double GAM_E = 4.0 / 3.0;
constexpr double KAPPA_MAX = 3.0;
constexpr double MP_ME = 1836.15267343;

// value of a scalar on the upwind side of the lower face (mass flux m) of the
// zone at offset c, zones st apart: the reconstruction of the zone below at its
// upper edge, or of the zone above at its lower edge, which is the same read in
// reverse order
template <int RECON>
__device__ inline double upwind(const double* E, int c, int st, double m) {
  const bool up = m >= 0.0;
  auto at = [&](int lo, int hi) -> double {
    const double a = buf_at(E + lo * st, c), b = buf_at(E + hi * st, c);
    return up ? a : b;
  };
  if (RECON == GRMHD_RECON_MC) {
    const double a = at(-2, 1), b = at(-1, 0), e = at(0, -1);
    return McSlope<double>(b - a, e - b).above(b);
  }
  return weno5_edge(at(-3, 2), at(-2, 1), at(-1, 0), at(0, -1), at(1, -2));
}

// r43: rho^(4/3)
__device__ double heating_fraction(int model, double fel, double rho, double r43, double u, double kel, double bsq,
                                   double gam) {
  if (model == GRMHD_HEAT_CONSTANT) return fel;
  const double pg = (gam - 1.0) * u;
  const double pe = kel * r43;
  const double pi = fmax(pg - pe, 1e-30 * pg + 1e-300);
  const double pb = 0.5 * bsq + 1e-300;
  const double beta = pi / pb;
  if (model == GRMHD_HEAT_KAWAZURA) {
    const double qi_qe = 35.0 / (1.0 + pow(beta / 15.0, -1.4) * exp(-0.1 * (pe / pi)));
    return 1.0 / (1.0 + qi_qe);
  }
  if (model == GRMHD_HEAT_WERNER) {
    const double s5 = bsq / rho / 5.0;
    return 0.25 * (1.0 + sqrt(s5 / (2.0 + s5)));
  }
  if (model == GRMHD_HEAT_ROWAN) {
    const double sw = bsq / (rho + u + pg);
    const double bmax = 1.0 / (4.0 * sw + 1e-300);
    const double x = fmax(1.0 - beta / bmax, 0.0);
    return 0.5 * exp(-pow(x, 3.3) / (1.0 + 1.2 * pow(sw, 0.7)));
  }
  if (model == GRMHD_HEAT_SHARMA) return 1.0 / (1.0 + 3.0 * sqrt(pi / fmax(pe, 1e-300)));
  // Howes
  const double theta = pi / fmax(pe, 1e-300);
  const double lt = log10(theta);
  const double c2 = (theta > 1.0 ? 1.6 : 1.2) / theta;
  const double c3 = theta > 1.0 ? 18.0 + 5.0 * lt : 18.0;
  const double x = 2.0 - 0.2 * lt;
  const double bx = exp(fmin(x * log(beta), 700.0));
  const double qi_qe = 0.92 * (c2 * c2 + bx) / (c3 * c3 + bx) * sqrt(MP_ME * theta) * exp(-1.0 / beta);
  return 1.0 / (1.0 + qi_qe);
}

// Advection and heating of a zone in one thread, with U_K, the metric and the
// zone's own entropies kept in registers between them: 0.27 ms on 288x128x128
// FP64 MC zones, against 0.39 ms for an advection and a heating kernel with U_K
// in memory. Of that, about 0.15 ms is arithmetic (1050 vector instructions a
// zone, pow and the model's transcendentals with them) and 0.17 ms the memory's
// copy rate; the 61 loads keep the address units 77 % busy. Neither 4 waves a
// SIMD (0.28 ms), the two entropies in turn with 86 registers (0.27 ms), nor the
// new state's loads first (0.27 ms) made it faster.
// b: block index within this job's grid (the update tile, XCD-aware order)
template <typename TF, int RECON>
__device__ void electron_body(const Dims& d, const double* __restrict__ cent, const UpdateParams& up,
                              const FluxOut<TF>& F, const double* Pb, double* P, const double* Eb, const double* Es, double* Eout,
                              double dt, int model, double fel, unsigned* bad, int b) {
  const TileK tk = xcd_tile_k(b, d.utx, d.uty, d.n1, d.n3);
  const int i = tk.i0 + (int)threadIdx.x;
  const int j = tk.j0 + (int)threadIdx.y;
  if (!tk.valid || i >= d.n1 || j >= d.n2) return;
  const int c = cell_of(d, tk.k, j, i);
  const size_t sv = (size_t)d.sv;
  const TF *m1 = F.m, *m2 = F.m + sv, *m3 = F.f3;  // mass fluxes
  const double f[6] = {(double)buf_at(m1, c),
                       (double)buf_at(m1 + 1, c),
                       up.polar_lo && j == 0 ? 0.0 : (double)buf_at(m2, c),
                       up.polar_hi && j == d.n2 - 1 ? 0.0 : (double)buf_at(m2 + d.s2, c),
                       (double)buf_at(m3, c),
                       (double)buf_at(m3 + d.s3, c)};
  ZoneGeo g;
  zone_geo<ZONE_ANY>(g, pair_plane(cent, d, tk.k), d, tab_of(d, j, i), i, j, tk.k);
  double Db;
  if (Pb) {
    const double v1 = buf_at(Pb + 2 * sv, c), v2 = buf_at(Pb + 3 * sv, c), v3 = buf_at(Pb + 4 * sv, c);
    double u1, u2, u3;
    lower3<false>(g, v1, v2, v3, u1, u2, u3);
    const double l2 = v1 * u1 + v2 * u2 + v3 * u3 + 1.0;
    Db = g.gdet * buf_at(Pb, c) * (l2 * rsqrt_full(l2) * g.ialpha);
    F.r[c] = Db;
  } else {
    Db = buf_at(F.r, c);
  }
  double uk[GRMHD_NSCALAR];
#pragma unroll
  for (int s = 0; s < GRMHD_NSCALAR; ++s) {
    const double* q = Es + s * sv;
    const double d1 = f[1] * upwind<RECON>(q + 1, c, 1, f[1]) - f[0] * upwind<RECON>(q, c, 1, f[0]);
    const double d2 = f[3] * upwind<RECON>(q + d.s2, c, d.s2, f[3]) - f[2] * upwind<RECON>(q, c, d.s2, f[2]);
    const double d3 = f[5] * upwind<RECON>(q + d.s3, c, d.s3, f[5]) - f[4] * upwind<RECON>(q, c, d.s3, f[4]);
    uk[s] = Db * buf_at(Eb + s * sv, c) - dt * (d1 * up.idx1 + d2 * up.idx2 + d3 * up.idx3);
  }
  const double gam = up.gam;
  double p[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) p[v] = buf_at(P + v * sv, c);
  const double rho = p[0];
  const double rg = pow(rho, gam);
  const double umax = KAPPA_MAX * rg / (gam - 1.0);
  if (p[1] > umax) {
    p[1] = umax;
    P[sv + c] = umax;
  }
  ZoneState st;
  zone_state<false>(p, g, st);
  const double iD = 1.0 / (g.gdet * rho * st.ut);
  const double ktot_adv = uk[0] * iD, kel_adv = uk[1] * iD;
  const double ktot = (gam - 1.0) * p[1] / rg;
  const double r43 = rho * cbrt(rho);
  const double fe = heating_fraction(model, fel, rho, r43, p[1], kel_adv, st.bsq, gam);
  const double scale = rg / r43;  // rho^(gam - 4/3)
  double kel = kel_adv + fe * (GAM_E - 1.0) / (gam - 1.0) * scale * (ktot - ktot_adv);
  kel = fmin(fmax(kel, 0.0), scale * ktot);
  Eout[c] = ktot;
  Eout[sv + c] = kel;
  if (!(isfinite(ktot) && isfinite(kel))) atomicAdd(bad, 1u);
}

template <typename TF, int RECON>
__global__ __launch_bounds__(256) void electron_kernel(Dims d, const double* __restrict__ cent, UpdateParams up,
                                                       FluxOut<TF> F, const double* Pb, double* P,
                                                       const double* Eb, const double* Es, double* Eout, double dt, const double* __restrict__ dt_dev,
                                                       double dt_scale, int model, double fel, Counters* ctr) {
  if (dt_dev) dt = dt_scale * *dt_dev;
  electron_body<TF, RECON>(d, cent, up, F, Pb, P, Eb, Es, Eout, dt, model, fel, &ctr->bad, (int)blockIdx.x);
}

// every job with entropies in one grid: predictor (fluxes of E, base E) into
// E_h, corrector (fluxes of E_h, base E) into E
template <typename TF, int RECON>
__global__ __launch_bounds__(256) void electron_batch_kernel(BatchView bv, int corrector) {
  const int* offs = bv.offs + PH_UPDATE * (bv.njobs + 1);
  const int jb = batch_job(offs, bv.njobs, (int)blockIdx.x);
  const JobDesc& J = bv.jobs[jb];
  if (!J.E) return;
  const double dt = corrector ? *J.dt : 0.5 * *J.dt;
  electron_body<TF, RECON>(J.d, global_ptr(J.t.cent), J.up, flux_out<TF>(global_ptr((unsigned char*)J.F), J.d.sv),
                           corrector ? nullptr : global_ptr(J.P), global_ptr(corrector ? J.P : J.Ph), global_ptr(J.E), global_ptr(corrector ? J.Eh : J.E),
                           global_ptr(corrector ? J.E : J.Eh), dt, J.heat_model, J.fel, global_ptr(&J.ctr->bad),
                           (int)blockIdx.x - offs[jb]);
}

template <typename TF, int RECON>
void electrons_for(const Dims& d, const Tables& t, const UpdateParams& up, const void* F, const double* Pb, double* P, const double* Eb,
                   const double* Es, double* Eout, double dt, const double* dt_dev, double dt_scale, int model,
                   double fel, Counters* ctr, hipStream_t s) {
  const dim3 grid(xcd_grid(d.n1, d.n2, d.n3, d.utx, d.uty)), block(d.utx, d.uty, 1);
  hipLaunchKernelGGL((electron_kernel<TF, RECON>), grid, block, 0, s, d, t.cent, up,
                     flux_out<TF>((unsigned char*)F, d.sv), Pb, P, Eb, Es, Eout, dt, dt_dev, dt_scale, model, fel, ctr);
}

}  // namespace

hipError_t launch_electrons(bool mixed, int recon, const Dims& d, const Tables& t, const UpdateParams& up,
                            const void* F, const double* Pb, double* P, const double* Eb, const double* Es, double* Eout, double dt,
                            const double* dt_dev, double dt_scale, int model, double fel, Counters* ctr,
                            hipStream_t s) {
  const bool mc = recon == GRMHD_RECON_MC;
  const auto launch = mixed ? (mc ? electrons_for<float, GRMHD_RECON_MC> : electrons_for<float, GRMHD_RECON_WENO5>)
                            : (mc ? electrons_for<double, GRMHD_RECON_MC> : electrons_for<double, GRMHD_RECON_WENO5>);
  launch(d, t, up, F, Pb, P, Eb, Es, Eout, dt, dt_dev, dt_scale, model, fel, ctr, s);
  return hipGetLastError();
}

hipError_t launch_batch_electrons(const BatchView& bv, const int* totals, bool mixed, int recon, bool corrector,
                                  hipStream_t s) {
  const dim3 grid(totals[PH_UPDATE]), block(bv.utx, bv.uty, 1);
  const bool mc = recon == GRMHD_RECON_MC;
  const auto kernel =
      mixed ? (mc ? electron_batch_kernel<float, GRMHD_RECON_MC> : electron_batch_kernel<float, GRMHD_RECON_WENO5>)
            : (mc ? electron_batch_kernel<double, GRMHD_RECON_MC> : electron_batch_kernel<double, GRMHD_RECON_WENO5>);
  hipLaunchKernelGGL(kernel, grid, block, 0, s, bv, corrector ? 1 : 0);
  return hipGetLastError();
}
