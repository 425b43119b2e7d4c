// Cartesian Kerr-Schild geometry of a point in closed form, for the face
// tables, and for the kernels that compute it instead of reading it; and the
// geometry of a zone centre, wherever it comes from. Implementation Notes section: a change of coordinates or background
// spacetime only changes the metric evaluation. The metric is
// g = eta + f l l with f = 2 r^3 / (r^4 + a^2 z^2) and the covector
// l = (1, (r x + a y)/(r^2 + a^2), (r y - a x)/(r^2 + a^2), z/r), null for
// both eta and g; hence g^-1 = eta - f l^ l^ with l^ = (-1, l1, l2, l3),
// det g = -1 (sqrt(-g) = 1) and the lapse 1/sqrt(-g^tt) = 1/sqrt(1 + f).
// Both users evaluate the same operations without contraction, so the values
// are the same bits wherever they come from.
#pragma once

#include "common.h"

// on the host, so that every user of the box has the same bits
inline CksBox cks_box(const grmhd_problem& p) {
  CksBox b;
  b.x0[0] = p.x1min;
  b.x0[1] = p.x2min;
  b.x0[2] = p.x3min;
  b.dx[0] = (p.x1max - p.x1min) / p.n1;
  b.dx[1] = (p.x2max - p.x2min) / p.n2;
  b.dx[2] = (p.x3max - p.x3min) / p.n3;
  b.a = p.a;
  return b;
}

// the positive root r of r^4 - (R^2 - a^2) r^2 - a^2 z^2 = 0, R^2 = x^2 + y^2 + z^2
__device__ inline double cks_radius(double x, double y, double z, double a) {
#pragma clang fp contract(off)
  const double h = 0.5 * (x * x + y * y + z * z - a * a);
  return sqrt(h + sqrt(h * h + a * a * z * z));
}

// f and l_i at (x, y, z)
__device__ inline void cks_null(double x, double y, double z, double a, double& f, double& l1, double& l2, double& l3) {
#pragma clang fp contract(off)
  const double h = 0.5 * (x * x + y * y + z * z - a * a);
  const double r = sqrt_full(h + sqrt_full(h * h + a * a * z * z));
  const double r2 = r * r;
  f = 2.0 * r2 * r * rcp_full(r2 * r2 + a * a * z * z);
  const double ira = rcp_full(r2 + a * a);
  l1 = (r * x + a * y) * ira;
  l2 = (r * y - a * x) * ira;
  l3 = z * rcp_full(r);
}

// step of the centred differences of the metric
constexpr double FD_DELTA = 1e-5;

// g_mn at (x, y, z) in the symmetric order, by the operations of its formula
// one by one (the difference quotients multiply a last-place change by 1e5)
__device__ inline void cks_gcov(double x, double y, double z, double a, double* g) {
#pragma clang fp contract(off)
  const double h = 0.5 * (x * x + y * y + z * z - a * a);
  const double r = sqrt_full(h + sqrt_full(h * h + a * a * z * z));
  const double r2 = r * r;
  const double fd = r2 * r2 + a * a * z * z, ra = r2 + a * a;
  const double f = div_by(2.0 * r2 * r, fd, rcp_full(fd));
  const double ira = rcp_full(ra);
  const double l1 = div_by(r * x + a * y, ra, ira), l2 = div_by(r * y - a * x, ra, ira), l3 = div_by(z, r, rcp_full(r));
  const double f1 = f * l1, f2 = f * l2, f3 = f * l3;
  g[0] = f - 1.0;
  g[1] = f1;
  g[2] = f2;
  g[3] = f3;
  g[4] = f1 * l1 + 1.0;
  g[5] = f1 * l2;
  g[6] = f1 * l3;
  g[7] = f2 * l2 + 1.0;
  g[8] = f2 * l3;
  g[9] = f3 * l3 + 1.0;
}

// at the lower D-face (D = 1..3) of cell (i, j, k), in the 3+1 form of the face
// tables: g_ij = delta_ij + f l_i l_j, alpha^2 = 1/(1 + f), beta^i = alpha^2 f
// l_i, gamma^ij = delta_ij - alpha^2 f l_i l_j
__device__ inline void cks_face_geo(const CksBox& b, int D, int i, int j, int k, FaceGeo<double>& g) {
#pragma clang fp contract(off)
  const double x = b.x0[0] + (D == 1 ? (double)i : i + 0.5) * b.dx[0];
  const double y = b.x0[1] + (D == 2 ? (double)j : j + 0.5) * b.dx[1];
  const double z = b.x0[2] + (D == 3 ? (double)k : k + 0.5) * b.dx[2];
  double f, l1, l2, l3;
  cks_null(x, y, z, b.a, f, l1, l2, l3);
  const double f1 = f * l1, f2 = f * l2, f3 = f * l3;
  const double al = rsqrt_full(1.0 + f), ia = (1.0 + f) * al, a2 = al * al;
  g.g11 = f1 * l1 + 1.0;
  g.g12 = f1 * l2;
  g.g13 = f1 * l3;
  g.g22 = f2 * l2 + 1.0;
  g.g23 = f2 * l3;
  g.g33 = f3 * l3 + 1.0;
  g.alpha = al;
  g.ialpha = ia;
  g.b1 = a2 * f1;
  g.b2 = a2 * f2;
  g.b3 = a2 * f3;
  g.H = a2 * (1.0 - (D == 1 ? g.b1 * l1 : D == 2 ? g.b2 * l2 : g.b3 * l3));
  g.hgdet = 0.5;
}

// the centre of cell (i, j, k), and the geometry there
__device__ inline void cks_centre(const CksBox& b, int i, int j, int k, double* x) {
#pragma clang fp contract(off)
  x[0] = b.x0[0] + (i + 0.5) * b.dx[0];
  x[1] = b.x0[1] + (j + 0.5) * b.dx[1];
  x[2] = b.x0[2] + (k + 0.5) * b.dx[2];
}
__device__ inline void cks_centre_geo(const CksBox& b, int i, int j, int k, ZoneGeo& g) {
#pragma clang fp contract(off)
  double c[3];
  cks_centre(b, i, j, k, c);
  const double x = c[0], y = c[1], z = c[2];
  double f, l1, l2, l3;
  cks_null(x, y, z, b.a, f, l1, l2, l3);
  const double f1 = f * l1, f2 = f * l2, f3 = f * l3;
  const double al = rsqrt_full(1.0 + f), ia = (1.0 + f) * al, a2 = al * al;
  g.g11 = f1 * l1 + 1.0;
  g.g12 = f1 * l2;
  g.g13 = f1 * l3;
  g.g22 = f2 * l2 + 1.0;
  g.g23 = f2 * l3;
  g.g33 = f3 * l3 + 1.0;
  g.alpha = al;
  g.ialpha = ia;
  g.b1 = a2 * f1;
  g.b2 = a2 * f2;
  g.b3 = a2 * f3;
  g.h11 = 1.0 - g.b1 * l1;
  g.h12 = -g.b1 * l2;
  g.h13 = -g.b1 * l3;
  g.h22 = 1.0 - g.b2 * l2;
  g.h23 = -g.b2 * l3;
  g.h33 = 1.0 - g.b3 * l3;
  g.gdet = 1.0;
  g.igdet = 1.0;
}

// The geometry of a zone: read from the table (MKS, FMKS, Minkowski; ct the
// plane of pair_plane, off the point of tab_of), evaluated (Cartesian
// Kerr-Schild), or whichever the context's coordinates call for.
enum { ZONE_AXI = 0, ZONE_CKS, ZONE_ANY };
__device__ inline double2 zone_pair(const double* ct, const Dims& d, int off, int c) {
  return buf_pair(ct + (size_t)c * d.ts, (unsigned)off * 16u);
}
template <int Z>
__device__ inline void zone_geo(ZoneGeo& g, const double* ct, const Dims& d, int off, int i, int j, int k) {
  if (Z == ZONE_CKS || (Z == ZONE_ANY && d.tk != 0)) {
    cks_centre_geo(d.box, i, j, k, g);
    return;
  }
  double2 q = zone_pair(ct, d, off, C_G11);
  g.g11 = q.x, g.g12 = q.y;
  q = zone_pair(ct, d, off, C_G13);
  g.g13 = q.x, g.g22 = q.y;
  q = zone_pair(ct, d, off, C_G33);
  g.g33 = q.x, g.alpha = q.y;
  q = zone_pair(ct, d, off, C_B1);
  g.b1 = q.x, g.b2 = q.y;
  q = zone_pair(ct, d, off, C_IALPHA);
  g.ialpha = q.x, g.gdet = q.y;
  q = zone_pair(ct, d, off, C_H11);
  g.h11 = q.x, g.h12 = q.y;
  q = zone_pair(ct, d, off, C_H13);
  g.h13 = q.x, g.h22 = q.y;
  q = zone_pair(ct, d, off, C_H23);
  g.h23 = q.x, g.h33 = q.y;
  g.igdet = zone_pair(ct, d, off, C_IGDET).x;
  g.g23 = 0.0;
  g.b3 = 0.0;
}
// rho_fl k and u_fl k^gamma
template <int Z>
__device__ inline void zone_floors(double& rfl, double& ufl, const double* ct, const Dims& d, int off) {
  if (Z == ZONE_CKS || (Z == ZONE_ANY && d.tk != 0)) {
    const double2 q = zone_pair(ct, d, off, K_RHOFL);
    rfl = q.x;
    ufl = q.y;
  } else {
    rfl = zone_pair(ct, d, off, C_RHOFL & ~1).y;
    ufl = zone_pair(ct, d, off, C_UFL).x;
  }
}
static_assert(!(K_RHOFL & 1) && K_UFL == K_RHOFL + 1 && (C_RHOFL & 1) && !(C_UFL & 1) && !(C_IGDET & 1), "pairs of the centre table");
