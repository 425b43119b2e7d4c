// Geometry tables: the metric in 3+1 form at zone centres and faces, the source
// coefficients (centred differences of the metric) and floor scales at centres
// (in Cartesian Kerr-Schild only floor scales: the kernels evaluate the rest).
// Implementation Notes section: every metric-dependent quantity is
// evaluated numerically from an analytic line element, the coordinates act as
// static mesh refinement (MKS / funky MKS concentrate zones towards the disk
// midplane), and another coordinate system or stationary spacetime is a small
// change: Cartesian Kerr-Schild (metric eta + f l l in (t, x, y, z)) makes
// every table depend on x3, so its tables are 3D with an x3-face table.
#include "kernels.h"
#include "cks_geometry.h"

// No fused multiply-adds here: the centred differences (step 1e-5) turn a
// one-ulp change of the metric into a 1e-10 change of its derivative, so
// every table value is the plain sequence of correctly rounded operations its
// formula spells out.
#pragma clang fp contract(off)

namespace {

constexpr double PI = 3.14159265358979323846;
constexpr double SIN_MIN = 1e-20;  // |sin theta| floor inside the metric (polar faces)

// theta(x1, x2) of MKS / funky MKS
__device__ double theta_of(double x1, double x2, const grmhd_problem& p) {
  const double tg = PI * x2 + 0.5 * (1.0 - p.hslope) * sin(2.0 * PI * x2);
  if (p.coords == GRMHD_KERR_MKS) return tg;
  const double al = p.poly_alpha, xt = p.poly_xt;
  const double norm = 0.5 * PI / (1.0 + 1.0 / ((al + 1.0) * pow(xt, al)));
  const double y = 2.0 * x2 - 1.0;
  const double tj = norm * y * (1.0 + pow(y / xt, al) / (al + 1.0)) + 0.5 * PI;
  return tg + exp(-p.mks_smooth * (x1 - p.x1min)) * (tj - tg);
}

__device__ void theta_derivs(double x1, double x2, const grmhd_problem& p, double& d1, double& d2) {
  const double dtg = PI * (1.0 + (1.0 - p.hslope) * cos(2.0 * PI * x2));
  if (p.coords == GRMHD_KERR_MKS) {
    d1 = 0.0;
    d2 = dtg;
    return;
  }
  const double tg = PI * x2 + 0.5 * (1.0 - p.hslope) * sin(2.0 * PI * x2);
  const double al = p.poly_alpha, xt = p.poly_xt;
  const double norm = 0.5 * PI / (1.0 + 1.0 / ((al + 1.0) * pow(xt, al)));
  const double y = 2.0 * x2 - 1.0;
  const double yp = pow(y / xt, al);
  const double tj = norm * y * (1.0 + yp / (al + 1.0)) + 0.5 * PI;
  const double dtj = 2.0 * norm * (1.0 + yp);
  const double e = exp(-p.mks_smooth * (x1 - p.x1min));
  d1 = -p.mks_smooth * e * (tj - tg);
  d2 = dtg + e * (dtj - dtg);
}

// covariant metric in MKS, FMKS or Minkowski coordinates, full 4x4
__device__ void gcov_code(double x1, double x2, const grmhd_problem& p, double g[4][4]) {
  for (int m = 0; m < 4; ++m)
    for (int n = 0; n < 4; ++n) g[m][n] = 0.0;
  if (p.coords == GRMHD_MINKOWSKI_CART) {
    g[0][0] = -1.0;
    g[1][1] = g[2][2] = g[3][3] = 1.0;
    return;
  }
  const double a = p.a;
  const double r = exp(x1);
  const double th = theta_of(x1, x2, p);
  double d1, d2;
  theta_derivs(x1, x2, p, d1, d2);
  double sth = sin(th);
  if (fabs(sth) < SIN_MIN) sth = SIN_MIN;
  const double s2 = sth * sth;
  const double cth = cos(th);
  const double rho2 = r * r + a * a * cth * cth;
  const double f = 2.0 * r / rho2;
  // Kerr-Schild (t, r, theta, phi)
  const double ktt = -(1.0 - f), ktr = f, ktp = -a * f * s2, krr = 1.0 + f;
  const double krp = -a * s2 * (1.0 + f), khh = rho2, kpp = s2 * (rho2 + a * a * s2 * (1.0 + f));
  // J: r = exp(x1) -> dr/dx1 = r; theta(x1, x2); phi = x3
  g[0][0] = ktt;
  g[0][1] = g[1][0] = ktr * r;
  g[0][3] = g[3][0] = ktp;
  g[1][1] = krr * r * r + khh * d1 * d1;
  g[1][2] = g[2][1] = khh * d1 * d2;
  g[1][3] = g[3][1] = krp * r;
  g[2][2] = khh * d2 * d2;
  g[3][3] = kpp;
}

// inverse and determinant by expansion in complementary 2x2 minors
__device__ double invert4(const double m[4][4], double b[4][4]) {
  const double s0 = m[0][0] * m[1][1] - m[1][0] * m[0][1];
  const double s1 = m[0][0] * m[1][2] - m[1][0] * m[0][2];
  const double s2 = m[0][0] * m[1][3] - m[1][0] * m[0][3];
  const double s3 = m[0][1] * m[1][2] - m[1][1] * m[0][2];
  const double s4 = m[0][1] * m[1][3] - m[1][1] * m[0][3];
  const double s5 = m[0][2] * m[1][3] - m[1][2] * m[0][3];
  const double c5 = m[2][2] * m[3][3] - m[3][2] * m[2][3];
  const double c4 = m[2][1] * m[3][3] - m[3][1] * m[2][3];
  const double c3 = m[2][1] * m[3][2] - m[3][1] * m[2][2];
  const double c2 = m[2][0] * m[3][3] - m[3][0] * m[2][3];
  const double c1 = m[2][0] * m[3][2] - m[3][0] * m[2][2];
  const double c0 = m[2][0] * m[3][1] - m[3][0] * m[2][1];
  const double det = s0 * c5 - s1 * c4 + s2 * c3 + s3 * c2 - s4 * c1 + s5 * c0;
  const double id = 1.0 / det;
  b[0][0] = (m[1][1] * c5 - m[1][2] * c4 + m[1][3] * c3) * id;
  b[0][1] = (-m[0][1] * c5 + m[0][2] * c4 - m[0][3] * c3) * id;
  b[0][2] = (m[3][1] * s5 - m[3][2] * s4 + m[3][3] * s3) * id;
  b[0][3] = (-m[2][1] * s5 + m[2][2] * s4 - m[2][3] * s3) * id;
  b[1][0] = (-m[1][0] * c5 + m[1][2] * c2 - m[1][3] * c1) * id;
  b[1][1] = (m[0][0] * c5 - m[0][2] * c2 + m[0][3] * c1) * id;
  b[1][2] = (-m[3][0] * s5 + m[3][2] * s2 - m[3][3] * s1) * id;
  b[1][3] = (m[2][0] * s5 - m[2][2] * s2 + m[2][3] * s1) * id;
  b[2][0] = (m[1][0] * c4 - m[1][1] * c2 + m[1][3] * c0) * id;
  b[2][1] = (-m[0][0] * c4 + m[0][1] * c2 - m[0][3] * c0) * id;
  b[2][2] = (m[3][0] * s4 - m[3][1] * s2 + m[3][3] * s0) * id;
  b[2][3] = (-m[2][0] * s4 + m[2][1] * s2 - m[2][3] * s0) * id;
  b[3][0] = (-m[1][0] * c3 + m[1][1] * c1 - m[1][2] * c0) * id;
  b[3][1] = (m[0][0] * c3 - m[0][1] * c1 + m[0][2] * c0) * id;
  b[3][2] = (-m[3][0] * s3 + m[3][1] * s1 - m[3][2] * s0) * id;
  b[3][3] = (m[2][0] * s3 - m[2][1] * s1 + m[2][2] * s0) * id;
  return det;
}

// the 3+1 quantities of a face of direction D in MKS, FMKS or Minkowski
// coordinates, whose g_23 and beta^3 vanish identically
__device__ void face_point(double x1, double x2, int D, const grmhd_problem& p, FaceGeo<double>& f) {
  double g[4][4], gi[4][4];
  gcov_code(x1, x2, p, g);
  const double det = invert4(g, gi);
  const double a2 = -1.0 / gi[0][0];
  f.g11 = g[1][1];
  f.g12 = g[1][2];
  f.g13 = g[1][3];
  f.g22 = g[2][2];
  f.g23 = 0.0;
  f.g33 = g[3][3];
  f.alpha = sqrt(a2);
  f.ialpha = sqrt(-gi[0][0]);
  f.b1 = a2 * gi[0][1];
  f.b2 = a2 * gi[0][2];
  f.b3 = 0.0;
  // gamma^DD by cofactors of g_ij
  const double c11 = f.g22 * f.g33, c22 = f.g11 * f.g33 - f.g13 * f.g13, c33 = f.g11 * f.g22 - f.g12 * f.g12;
  const double d3 = f.g33 * c33 - f.g13 * f.g13 * f.g22;
  f.H = a2 * ((D == 1 ? c11 : D == 2 ? c22 : c33) / d3);
  f.hgdet = 0.5 * sqrt(fabs(det));
}

// a face table entry (paired components) and its float copy
__device__ void store_face(const FaceGeo<double>& g, double* dt, float* ft, size_t ts, int off) {
  double v[F_USED] = {};
  v[F_G11] = g.g11;
  v[F_G12] = g.g12;
  v[F_G13] = g.g13;
  v[F_G22] = g.g22;
  v[F_G33] = g.g33;
  v[F_ALPHA] = g.alpha;
  v[F_B1] = g.b1;
  v[F_B2] = g.b2;
  v[F_IALPHA] = g.ialpha;
  v[F_H] = g.H;
  v[F_HGDET] = g.hgdet;
  v[F_B3] = g.b3;
  v[F_G23] = g.g23;
  for (int c = 0; c < F_USED; ++c) {
    dt[pair_index(c, ts, (size_t)off)] = v[c];
    ft[pair_index(c, ts, (size_t)off)] = (float)v[c];
  }
}

__global__ void geometry_kernel(grmhd_problem p, Dims d, Tables t) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x) - NG;
  const int j = (int)(blockIdx.y * blockDim.y + threadIdx.y) - NG;
  const int k = (int)blockIdx.z - NG;  // 2D tables: a single plane (k = -NG, tk = 0)
  if (i >= d.n1 + NG || j >= d.n2 + NG) return;
  const int off = (k + NG) * d.tk + tab_of(d, j, i);
  const size_t ts = (size_t)d.ts;
  const double dx1 = (p.x1max - p.x1min) / p.n1;
  const double dx2 = (p.x2max - p.x2min) / p.n2;
  const double dx3 = (p.x3max - p.x3min) / p.n3;
  const double x1c = p.x1min + (i + 0.5) * dx1, x2c = p.x2min + (j + 0.5) * dx2, x3c = p.x3min + (k + 0.5) * dx3;
  const double x1f = p.x1min + i * dx1, x2f = p.x2min + j * dx2;
  const bool k3 = p.coords == GRMHD_KERR_CKS;
  const CksBox& box = d.box;  // the zone corner and widths, computed on the host

  // faces: Cartesian Kerr-Schild in closed form, the values the face-flux pass
  // computes itself (box: the zone corner and widths it uses, computed on the
  // host); the x3-face table of the 2D tables holds the centre values, the
  // metric not depending on x3
  double* const dt[3] = {t.f1, t.f2, t.f3};
  float* const ft[3] = {t.f1f, t.f2f, t.f3f};
  for (int D = 1; D <= 3; ++D) {
    FaceGeo<double> g;
    if (k3) cks_face_geo(box, D, i, j, k, g);
    else face_point(D == 1 ? x1f : x1c, D == 2 ? x2f : x2c, D, p, g);
    store_face(g, dt[D - 1], ft[D - 1], ts, off);
  }

  // centres
  double v[N_CENT] = {};
  int nc = C_UFL + 1;
  // floor scales: k = 1/(r^2 (1 + r/10)) with r = exp(x1) (MKS / FMKS) or the
  // Kerr-Schild radius of the Cartesian point
  double rfl = 0.0, ufl = 0.0;
  if (p.coords != GRMHD_MINKOWSKI_CART) {
    const double r = k3 ? cks_radius(x1c, x2c, x3c, p.a) : exp(x1c);
    const double kk = 1.0 / (r * r * (1.0 + r / 10.0));
    rfl = p.rho_fl * kk;
    ufl = p.u_fl * pow(kk, p.gam);
  }
  if (k3) {
    nc = K_GDET + 1;
    v[K_RHOFL] = rfl;
    v[K_UFL] = ufl;
    v[K_GDET] = 1.0;
  } else {
    double g[4][4], gi[4][4];
    gcov_code(x1c, x2c, p, g);
    const double det = invert4(g, gi);
    const double a2 = -1.0 / gi[0][0], gdet = sqrt(fabs(det));
    v[C_G11] = g[1][1];
    v[C_G12] = g[1][2];
    v[C_G13] = g[1][3];
    v[C_G22] = g[2][2];
    v[C_G33] = g[3][3];
    v[C_ALPHA] = 1.0 / sqrt(-gi[0][0]);
    v[C_B1] = a2 * gi[0][1];
    v[C_B2] = a2 * gi[0][2];
    v[C_IALPHA] = sqrt(-gi[0][0]);
    v[C_GDET] = gdet;
    v[C_IGDET] = 1.0 / gdet;
    // gamma^ij = g^ij + alpha^2 g^ti g^tj
    v[C_H11] = gi[1][1] + a2 * gi[0][1] * gi[0][1];
    v[C_H12] = gi[1][2] + a2 * gi[0][1] * gi[0][2];
    v[C_H13] = gi[1][3];
    v[C_H22] = gi[2][2] + a2 * gi[0][2] * gi[0][2];
    v[C_H23] = gi[2][3];
    v[C_H33] = gi[3][3];
    v[C_RHOFL] = rfl;
    v[C_UFL] = ufl;
    // source coefficients from centred differences of the metric in x1 and x2
    for (int c = 0; c < 2 && p.coords != GRMHD_MINKOWSKI_CART; ++c) {
      const double e1 = c == 0 ? FD_DELTA : 0.0, e2 = c == 1 ? FD_DELTA : 0.0;
      double gp[4][4], gm[4][4];
      gcov_code(x1c + e1, x2c + e2, p, gp);
      gcov_code(x1c - e1, x2c - e2, p, gm);
      double tr = 0.0;
      for (int q = 0; q < 8; ++q) {
        const int a = AXI_KM[q][0], b = AXI_KM[q][1];
        const double dg = gdet * ((gp[a][b] - gm[a][b]) / (2.0 * FD_DELTA)) * (a == b ? 0.5 : 1.0);
        tr += gi[a][b] * dg;
        v[C_S1 + 9 * c + q] = dg;
      }
      v[C_S1 + 9 * c + 8] = tr;
    }
  }
  for (int c = 0; c < nc; ++c) t.cent[pair_index(c, ts, (size_t)off)] = v[c];
}

}  // namespace

hipError_t launch_geometry(const grmhd_problem& p, const Dims& d, const Tables& t, hipStream_t s) {
  dim3 blk(64, 4, 1);
  dim3 grd((d.n1 + 2 * NG + 63) / 64, (d.n2 + 2 * NG + 3) / 4, d.tk ? d.p3 : 1);
  hipLaunchKernelGGL(geometry_kernel, grd, blk, 0, s, p, d, t);
  return hipGetLastError();
}
