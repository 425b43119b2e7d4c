// Face fluxes of all three directions, their divergence and the Flux-CT edge
// EMFs in one pass: reconstruct the primitives at the lower d-face of each zone
// (MC or WENO5), evaluate both face states (flux, conserved variables, fast-
// magnetosonic speeds), combine them with the local Lax-Friedrichs flux
//   F = (F_L + F_R)/2 - ctop (U_R - U_L)/2,
//   ctop = max(max(0, c+_L, c+_R), max(0, -c-_L, -c-_R)),
// and keep what the update needs of them: the divergence of the five
// hydrodynamic fluxes and the three EMFs of the zone's lower edges.
// Functionality section: HARM updates conserved variables by finite volumes;
// the reconstruction and Riemann solver follow the HARM literature. Flux-CT:
// Implementation Notes, after Toth 2000.
//
// Cells covered: faces 0..n_d along d, transverse indices -1..n_t (the extra
// transverse layer feeds the EMFs). A block holds a tile of (x1, x2) cells of
// one x3 plane, one thread per cell. It stages the plane's primitives with the
// stencil halo in LDS (the x1 and x2 stencils come from there, the rest of the
// x3 stencil from the state) and computes the x3, x1 and x2 face of each cell.
// The x1 neighbours' fluxes come from the next and previous lane (a row of the
// tile lies within a wave), the x2 neighbours' through LDS. A cell's divergence
// needs the next thread of its row and the next row, its EMFs and x1 face the
// previous ones, so neighbouring tiles overlap by two columns and one row; what needs the plane above
// or below (the x3 fluxes, the x1 and x2 flux of B3) goes out as it is.
//
// What bounds it: FP64 issue and the latency of its loads, about half each (a
// wave issues 1260 VALU instructions, 1410 with the Courant maxima, 480 of them the
// MC slopes). It runs
// at four waves a SIMD, so a face may hold 128 registers: sums and speeds wait
// in LDS, and FACE_FENCE keeps the three faces apart. On the 288 x 128 x 128
// torus in FP64 with MC slopes it takes 0.401 ms, 0.415 with the maxima. Writing
// the three flux arrays it took 0.451 where this form took 0.410, and the update,
// which then read 66 of their values a cell and now reads 35, 0.605 against 0.470
// (0.361 with its later changes; mixed-precision WENO5: the pass 0.50 -> 0.55, now
// 0.48, the update 0.57 -> 0.42, now 0.31). The tiles are walked x2 first, so a block finds the
// rows it shares with the tile before in the XCD's L2 (0.94 -> 0.61 GB read).
// A block that walks along 4 to 32 planes with running sums writes 8 values a
// cell instead of 15, but its registers leave three waves a SIMD and its
// geometry falls out of the L2 between planes: 0.50 ms.
//
// The face states are written in the 3+1 form (side_speeds, side_flux): 12 or
// 14 geometry values a face. WENO5 is bound by its arithmetic (2800 VALU
// instructions a wave in mixed precision before x2 shared its edges). In x1 a
// lane finds both edges of its own zone, which share the smoothness indicators
// (MC: the slope), and passes the right one on, in x2 a row does (row_sides);
// with the indicators in differences and one corrected reciprocal per division
// the pass takes 0.48 ms on the benchmark torus in mixed precision (0.55 with
// the plain formula at every face) and 88 us on 131 x 67 x 45 in FP64 (117).
//
// The per-direction maximum of ctop over the faces with interior transverse
// index feeds the Courant step (one atomic max per block and direction); a
// face with a NaN speed counts as +inf there, which the step reports as a
// non-finite state. The face geometry comes from the face tables, or for
// Cartesian Kerr-Schild in FP64 from its closed form (the same bits).
#include <atomic>
#include <type_traits>

#include "cks_geometry.h"
#include "kernels.h"

// Keeps one face's arithmetic out of the next one's: interleaved, the three
// faces of a cell need more registers than four waves a SIMD leave.
#define FACE_FENCE do { asm volatile("" ::: "memory"); __builtin_amdgcn_sched_barrier(0); } while (0)

namespace {

// source of the face geometry: a table of coordinates with g_23 = beta^3 = 0
// (MKS, FMKS, Minkowski), a general table, or the closed form of Cartesian
// Kerr-Schild (the bits of its table)
enum { GEO_AXI = 0, GEO_TABLE, GEO_CKS };

// the block's x3 plane of primitives with the stencil halo in x1 and x2,
// [8][lh][lw] of T, cells (ib + li, jb + lj)
// The block shape is a template parameter: the row length and the distance
// between variables are then constants, and a stencil read needs no address of
// its own per variable (with runtime strides the loop over planes kept some 50
// such addresses in registers and spilled).
template <int RECON, int BX_, int BY_>
struct PlaneShape {
  // halo: zones before / after the cell in x1 (both edges of the zone are found together) and
  // below / above it in x2 (the faces of a row need the zones below)
  static constexpr int LX = RECON == GRMHD_RECON_MC ? 1 : 2, HX = LX;
  static constexpr int LY = RECON == GRMHD_RECON_MC ? 2 : 3, HY = LY - 1;
  static constexpr int BX = BX_, BY = BY_;
  static constexpr int LW = BX + LX + HX, LH = BY + LY + HY, PLANE = LW * LH, NTHR = BX * BY;
};

// the value a lane's neighbour holds: the next lane of the wave, or the
// previous one (every lane of the wave must be active)
template <int CTRL>
__device__ inline int dpp32(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false); }
constexpr int WAVE_SHL1 = 0x130, WAVE_SHR1 = 0x138;
template <int CTRL>
__device__ inline float dpp(float x) { return __int_as_float(dpp32<CTRL>(__float_as_int(x))); }
template <int CTRL>
__device__ inline double dpp(double x) {
  return __hiloint2double(dpp32<CTRL>(__double2hiint(x)), dpp32<CTRL>(__double2loint(x)));
}
template <typename T>
__device__ inline T next_lane(T x) { return dpp<WAVE_SHL1>(x); }
template <typename T>
__device__ inline T prev_lane(T x) { return dpp<WAVE_SHR1>(x); }

// both edges, along the direction whose zones are st apart, of the zone at e:
// they share its slope or its smoothness indicators
template <int RECON, typename T>
__device__ inline void zone_edges(const T* e, int st, T& left, T& right) {
  if constexpr (RECON == GRMHD_RECON_MC) {
    const T c = e[0];
    const McSlope<T> m(c - e[-st], e[st] - c);
    left = m.below(c);
    right = m.above(c);
  } else {
    weno5_edges(e[-2 * st], e[-st], e[0], e[st], e[2 * st], left, right);
  }
}

// both sides of the lower D-face of the cell whose place in the staged plane
// is q; the other planes of an x3 stencil come from the state, at byte offset cb
// of each variable (planes pb apart), or, MC only, from z (planes -2, -1 and 1 of each
// variable) when it is not null
template <int D, int RECON, typename T, typename SH>
__device__ inline void face_sides(const double* __restrict__ P, size_t sv, const T* q, unsigned cb, unsigned pb,
                                  FaceSide<T>& L, FaceSide<T>& R, const double* z = nullptr) {
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const T* ql = q + v * SH::PLANE;
    if constexpr (D == 1) {
      // the left side of the cell's lower face is the right edge of the zone the lane before
      // holds (a row's first lane has none: its face is not used)
      T right;
      zone_edges<RECON>(ql, 1, R.P[v], right);
      L.P[v] = prev_lane(right);
      continue;
    }
    constexpr int st = SH::LW;
    // the cell's own value from the LDS tile in every direction
    auto at = [&](int o) -> T {
      if (D == 3 && o != 0 && z) return (T)z[3 * v + (o < 0 ? o + 2 : 2)];
      return (D == 3 && o != 0) ? (T)buf_f64(P + v * sv, cb + (unsigned)o * pb) : ql[o * st];
    };
    if constexpr (RECON == GRMHD_RECON_MC) {
      const T a = at(-2), bb = at(-1), e = at(0), f = at(1);
      const T dl = bb - a, dc = e - bb, dr = f - e;
      L.P[v] = McSlope<T>(dl, dc).above(bb);
      R.P[v] = McSlope<T>(dc, dr).below(e);
    } else {
      const T x0 = at(-3), x1 = at(-2), x2 = at(-1), x3 = at(0), x4 = at(1), x5 = at(2);
      L.P[v] = weno5_edge(x0, x1, x2, x3, x4);
      R.P[v] = weno5_edge(x5, x4, x3, x2, x1);
    }
  }
}

// Both sides of the lower x2-face of each cell: a row finds both edges of its
// own zones and hands the upper ones to the row above through LDS, over the
// staged plane (its last use). The first row's wave also finds those of the
// zones below, which wait in free, of 8 BX values. All threads of the block
// take part. WENO5 only: 0.488 -> 0.470 ms on the benchmark torus in mixed
// precision, 90 -> 88 us on 131 x 67 x 45 in FP64; an MC slope costs less than
// its way through LDS (0.404 -> 0.406 ms in FP64, mixed 58 -> 60 us on
// 160 x 96 x 48).
template <int RECON, typename T, typename SH>
__device__ inline void row_sides(T* plane, T* free, const T* q, int li, int lj, int tid, FaceSide<T>& L, FaceSide<T>& R) {
  constexpr int BX = SH::BX, ST = SH::NTHR + BX;  // rows -1..BY-1
  static_assert(NV * ST <= NV * SH::PLANE, "the exchanged rows fit the staged plane");
  const bool first = __builtin_amdgcn_readfirstlane(tid) < 64;
  if (first) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      T lo, hi;
      zone_edges<RECON>(q + v * SH::PLANE - SH::LW, SH::LW, lo, hi);
      if (lj == 0) free[v * BX + li] = hi;
      FACE_FENCE;
    }
  }
  FACE_FENCE;
  T up[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) zone_edges<RECON>(q + v * SH::PLANE, SH::LW, R.P[v], up[v]);
  __syncthreads();
  T* const x = plane + BX + tid;
#pragma unroll
  for (int v = 0; v < NV; ++v) x[v * ST] = up[v];
  if (lj == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v * ST - BX] = free[v * BX + li];
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; ++v) L.P[v] = x[v * ST - BX];
}

// Signal speeds of both sides of a face and their largest, ctop. CTOP: *top
// takes it for the Courant maximum, 0 for a face outside it (inner false) and
// +inf when a speed is not finite (fmax drops a NaN operand, so such a face
// would report a finite, often zero, speed)
template <int D, bool AXI, bool CTOP, typename T>
__device__ inline T face_speeds(FaceSide<T>& L, FaceSide<T>& R, const FaceGeo<T>& g, T gam, T* top, bool inner) {
  side_speeds<D, AXI>(L, g, gam);
  side_speeds<D, AXI>(R, g, gam);
  const T ct = fmax(fmax(fmax(T(0), L.cp), R.cp), fmax(-L.cm, -R.cm));
  if (CTOP) {
    const T chk = (L.cp + L.cm) + (R.cp + R.cm);
    *top = !inner ? T(0) : chk == chk ? ct : (T)__builtin_inf();
  }
  return ct;
}

// The local Lax-Friedrichs flux of a face (mass, energy, 3 momenta, then the
// two transverse field components in ascending order) in f
template <int D, bool AXI, bool CTOP, typename T>
__device__ inline void face_flux(FaceSide<T>& L, FaceSide<T>& R, const FaceGeo<T>& g, T gam, T* f, T* top, bool inner) {
  const T ct = face_speeds<D, AXI, CTOP>(L, R, g, gam, top, inner);
  T fr[7];
  side_flux<D, AXI>(L, g, gam, ct, f);
  side_flux<D, AXI>(R, g, gam, -ct, fr);
#pragma unroll
  for (int v = 0; v < 7; ++v) f[v] = g.hgdet * (f[v] + fr[v]);
}

// exchange through LDS between the rows of a tile: the x2 flux's five
// hydrodynamic components, the x1 flux of B2 and the x3 flux of B2
constexpr int NEXCH = 7;

// what a job's pass reads and writes
template <typename T>
struct SweepArgs {
  const double* P;
  const T *t1, *t2, *t3;
  FluxOut<T> out;
  T* mass;  // the three mass fluxes as well, for the electron entropies (null: not kept)
  double idx1, idx2, idx3;
  T gam;
  int polar_lo, polar_hi;
};

// stage the plane: cells [ib, ib + LW) x [jb, jb + LH), those inside the padded
// state (cells outside it are never read: faces start at cell 0 and end at n)
template <typename SH, typename T>
__device__ inline void stage_plane(const Dims& d, const double* P, T* L, int ib, int jb, int k, int tid) {
#pragma unroll
  for (int e0 = 0; e0 < SH::PLANE; e0 += SH::NTHR) {
    const int e = e0 + tid;
    const int ej = e / SH::LW, ei = e - ej * SH::LW;
    const int gi = ib + ei, gj = jb + ej;
    if (e < SH::PLANE && gi >= -NG && gi < d.n1 + NG && gj >= -NG && gj < d.n2 + NG) {
      const unsigned c = (unsigned)cell_of(d, k, gj, gi) * (unsigned)sizeof(double);
#pragma unroll
      for (int v = 0; v < NV; ++v) L[v * SH::PLANE + e] = (T)buf_f64(P + (size_t)v * d.sv, c);
    }
  }
}

// b: block index within this job's grid; BX x BY threads
template <int RECON, typename T, int GEO, bool CTOP, int BX, int BY>
__device__ void sweep_body(const Dims& d, const SweepArgs<T>& a, int b, unsigned long long* ctop) {
  using SH = PlaneShape<RECON, BX, BY>;
  const SweepTile t = sweep_tile(d, BX, BY, b);
  if (!t.valid) return;
  const int li = (int)threadIdx.x, lj = (int)threadIdx.y;
  const int i = t.i0 + li, j = t.j0 + lj, k = t.k;
  const bool ok = i <= d.n1 && j <= d.n2;
  extern __shared__ __align__(16) unsigned char sweep_lds[];
  T* const L = reinterpret_cast<T*>(sweep_lds);
  const T* const q = L + (lj + SH::LY) * SH::LW + li + SH::LX;
  const int tid = lj * BX + li;
  T* const X = L + NV * SH::PLANE + tid;  // this thread's slot of the exchange, [NEXCH][BY][BX]
  const int ib = t.i0 - SH::LX, jb = t.j0 - SH::LY;
  // the cells this thread writes: an x1 face needs the previous thread of the row, a divergence
  // the next one and the next row, an EMF the previous ones
  const bool wd = li > 0 && li < BX - 1 && i >= 0 && i < d.n1 && j >= 0 && j < d.n2 && lj < BY - 1;
  const int last = BX - 2 + (t.i0 + BX - 1 == d.n1);  // cell n may be the last column
  const bool we = li > 0 && li <= last && ok && i >= 0 && j >= 0 && lj > 0;
  const bool axis = (a.polar_lo && j == 0) || (a.polar_hi && j == d.n2);
  const bool in1 = i >= 0 && i < d.n1, in2 = j >= 0 && j < d.n2;
  // threads beyond the grid, and on faces no one asks for, compute on the nearest cell's data
  // and write nothing: no branch splits a face's arithmetic
  const int ic = min(i, d.n1), jc = min(j, d.n2);
  const unsigned pb = (unsigned)d.s3 * (unsigned)sizeof(double);
  const int toff = tab_of(d, jc, ic);
  constexpr bool AXI = GEO == GEO_AXI;
  const unsigned cb = (unsigned)cell_of(d, k, jc, ic) * (unsigned)sizeof(double);
  const size_t sv = (size_t)d.sv;
  stage_plane<SH>(d, a.P, L, ib, jb, k, tid);
  // Cartesian Kerr-Schild: the other planes' values are on their way while the
  // face's metric is evaluated (0.488 -> 0.466 ms on 168^3 zones; where the
  // metric is read, the registers cost more: 0.403 -> 0.406 on 288 x 128 x 128)
  constexpr bool AHEAD = RECON == GRMHD_RECON_MC && GEO == GEO_CKS;
  double z[AHEAD ? 3 * NV : 1];
  if constexpr (AHEAD) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      z[3 * v] = buf_f64(a.P + v * sv, cb - 2u * pb);
      z[3 * v + 1] = buf_f64(a.P + v * sv, cb - pb);
      z[3 * v + 2] = buf_f64(a.P + v * sv, cb + pb);
    }
  }
  __syncthreads();
  const int c = cell_of(d, k, j, i);
  const bool hydro = k >= 0 && k < d.n3;
  auto geo = [&](int D, const T* tab, FaceGeo<T>& g) {
    if constexpr (GEO == GEO_CKS) cks_face_geo(d.box, D, ic, jc, k, g);
    else load_face_geo<AXI>(g, pair_plane(tab, d, k), d.ts, toff);
  };
  T f[7];
  T g2 = T(0);  // x3 fluxes of B1 of this cell and the one before it
  if (k >= 0) {
    FaceGeo<T> g;
    geo(3, a.t3, g);
    FaceSide<T> SL, SR;
    face_sides<3, RECON, T, SH>(a.P, sv, q, cb, pb, SL, SR, AHEAD ? z : nullptr);
    // the speeds wait in slots that the exchange uses later
    face_flux<3, AXI, CTOP>(SL, SR, g, a.gam, f, X, in1 && in2);
    if (wd) {
#pragma unroll
      for (int v = 0; v < 5; ++v) a.out.f3[v * sv + c] = f[v];
    }
    g2 = f[5] + prev_lane(f[5]);
    X[6 * SH::NTHR] = f[6];
  }
  FACE_FENCE;
  double acc[5];
  {
    FaceGeo<T> g;
    geo(1, a.t1, g);
    FaceSide<T> SL, SR;
    face_sides<1, RECON, T, SH>(a.P, sv, q, cb, pb, SL, SR);
    face_flux<1, AXI, CTOP>(SL, SR, g, a.gam, f, X + SH::NTHR, li > 0 && ok && i >= 0 && in2 && hydro);
    // no mass enters through an outflow boundary: the rest-mass flux through
    // the inner radial face is at most 0, through the outer one at least 0
    if (d.out_lo && i == 0) f[0] = fmin(f[0], T(0));
    if (d.out_hi && i == d.n1) f[0] = fmax(f[0], T(0));
    if (a.mass && we && hydro) a.mass[c] = f[0];
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[v] = ((double)next_lane(f[v]) - (double)f[v]) * a.idx1;
    X[5 * SH::NTHR] = f[5];
    if (we) {
      a.out.b[sv + c] = f[6];
      if (k >= 0) a.out.e[sv + c] = g2 - f[6];
    }
  }
  FACE_FENCE;
  {
    FaceGeo<T> g;
    FaceSide<T> SL, SR;
    if constexpr (RECON == GRMHD_RECON_MC) {
      geo(2, a.t2, g);
      face_sides<2, RECON, T, SH>(a.P, sv, q, cb, pb, SL, SR);
    } else {
      // the exchange's fourth and fifth values are still free
      row_sides<RECON, T, SH>(L, L + NV * SH::PLANE + 3 * SH::NTHR, q, li, lj, tid, SL, SR);
      FACE_FENCE;
      geo(2, a.t2, g);
    }
    face_flux<2, AXI, CTOP>(SL, SR, g, a.gam, f, X + 2 * SH::NTHR, ok && j >= 0 && in1 && hydro);
    if (a.mass && we && hydro) a.mass[sv + c] = f[0];
    if (axis) {
#pragma unroll
      for (int v = 0; v < 5; ++v) f[v] = T(0);
      f[6] = T(0);
    }
  }
  FACE_FENCE;
  const T g3 = prev_lane(f[5]);
  double c1 = 0.0, c2 = 0.0, c3 = 0.0;
  if (CTOP) {
    if (k >= 0) c3 = (double)X[0];
    c1 = (double)X[SH::NTHR];
    c2 = (double)X[2 * SH::NTHR];
  }
  // rows exchange what the next and previous ones need
#pragma unroll
  for (int v = 0; v < 5; ++v) X[v * SH::NTHR] = f[v];
  __syncthreads();
  if (wd && hydro) {
#pragma unroll
    for (int v = 0; v < 5; ++v) a.out.D[v * sv + c] = fma(-((double)X[v * SH::NTHR + BX] - (double)f[v]), a.idx2, -acc[v]);
  }
  if (we) {
    a.out.b[c] = f[6];
    // four times the EMFs of the zone's lower edges (0 on a polar axis)
    if (hydro) a.out.e[2 * sv + c] = axis ? T(0) : ((X[5 * SH::NTHR] + X[5 * SH::NTHR - BX]) - f[5]) - g3;
    if (k >= 0) a.out.e[c] = axis ? T(0) : f[6] - (X[6 * SH::NTHR] + X[6 * SH::NTHR - BX]);
  }
  if (CTOP) block_max3_to(c1, c2, c3, ctop);
}

// At least four waves a SIMD in FP64, six in FP32 (three blocks a CU, as the LDS
// has it) and no more: left to aim at eight, the scheduler waits for each load of
// an x3 stencil before the next, 0.47 -> 0.52 ms on the benchmark torus with WENO5.
#define SWEEP_BOUNDS \
  __launch_bounds__(BX * BY) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 4 : 6, sizeof(T) == 8 ? 8 : 6)))

template <int RECON, typename T, int GEO, bool CTOP, int BX, int BY>
__global__ SWEEP_BOUNDS void sweep_kernel(Dims d, SweepArgs<T> a,
                                                                          unsigned long long* ctop) {
  sweep_body<RECON, T, GEO, CTOP, BX, BY>(d, a, (int)blockIdx.x, ctop);
}

// The Courant maxima alone, of a state whose fluxes no one asks for: the same
// tiles, faces and speeds, without flux, exchange or output (85 us on
// 192 x 96 x 64 FP64 MC zones, 117 to 122 with the fluxes). With WENO5 a row's
// edges cost 28 to 65 spilled registers in FP64, up to 8 in FP32; grmhd_get_dt
// takes 234 and 146 us there on that grid, 345 and 217 with the fluxes.
template <int RECON, typename T, int GEO, int BX, int BY>
__global__ __launch_bounds__(BX * BY, sizeof(T) == 8 ? 4 : 6) void speed_kernel(Dims d, SweepArgs<T> a,
                                                                          unsigned long long* ctop) {
  using SH = PlaneShape<RECON, BX, BY>;
  const SweepTile t = sweep_tile(d, BX, BY, (int)blockIdx.x);
  if (!t.valid || t.k < 0) return;
  const int li = (int)threadIdx.x, lj = (int)threadIdx.y, tid = lj * BX + li;
  const int i = t.i0 + li, j = t.j0 + lj, k = t.k;
  extern __shared__ __align__(16) unsigned char sweep_lds[];
  T* const L = reinterpret_cast<T*>(sweep_lds);
  const T* const q = L + (lj + SH::LY) * SH::LW + li + SH::LX;
  const bool ok = i <= d.n1 && j <= d.n2;
  const bool in1 = i >= 0 && i < d.n1, in2 = j >= 0 && j < d.n2, in3 = k < d.n3;
  const int ic = min(i, d.n1), jc = min(j, d.n2);
  const int toff = tab_of(d, jc, ic);
  const unsigned pb = (unsigned)d.s3 * (unsigned)sizeof(double);
  const unsigned cb = (unsigned)cell_of(d, k, jc, ic) * (unsigned)sizeof(double);
  const size_t sv = (size_t)d.sv;
  constexpr bool AXI = GEO == GEO_AXI;
  stage_plane<SH>(d, a.P, L, t.i0 - SH::LX, t.j0 - SH::LY, k, tid);
  __syncthreads();
  auto top = [&](auto dir, const T* tab, bool inner) -> double {
    constexpr int D = decltype(dir)::value;
    FaceSide<T> SL, SR;
    if constexpr (D == 2 && RECON != GRMHD_RECON_MC)
      row_sides<RECON, T, SH>(L, L + NV * SH::PLANE, q, li, lj, tid, SL, SR);
    else face_sides<D, RECON, T, SH>(a.P, sv, q, cb, pb, SL, SR);
    FACE_FENCE;
    FaceGeo<T> g;
    if constexpr (GEO == GEO_CKS) cks_face_geo(d.box, D, ic, jc, k, g);
    else load_face_geo<AXI>(g, pair_plane(tab, d, k), d.ts, toff);
    T m;
    face_speeds<D, AXI, true>(SL, SR, g, a.gam, &m, inner);
    double c = (double)m;
    asm volatile("" : "+v"(c));  // the face ends here
    FACE_FENCE;
    return c;
  };
  const double c3 = top(std::integral_constant<int, 3>(), a.t3, in1 && in2);
  const double c1 = top(std::integral_constant<int, 1>(), a.t1, li > 0 && ok && i >= 0 && in2 && in3);
  const double c2 = top(std::integral_constant<int, 2>(), a.t2, ok && j >= 0 && in1 && in3);
  block_max3_to(c1, c2, c3, ctop);
}

template <typename T>
struct FaceTables;
template <>
struct FaceTables<double> {
  __host__ __device__ static const double* f1(const Tables& t) { return t.f1; }
  __host__ __device__ static const double* f2(const Tables& t) { return t.f2; }
  __host__ __device__ static const double* f3(const Tables& t) { return t.f3; }
};
template <>
struct FaceTables<float> {
  __host__ __device__ static const float* f1(const Tables& t) { return t.f1f; }
  __host__ __device__ static const float* f2(const Tables& t) { return t.f2f; }
  __host__ __device__ static const float* f3(const Tables& t) { return t.f3f; }
};

// every job of a batch in one grid; predictor sweeps P, corrector sweeps P_h
template <int RECON, typename T, int GEO, bool CTOP, int BX, int BY>
__global__ SWEEP_BOUNDS void sweep_batch_kernel(BatchView bv, int corrector) {
  const int* offs = bv.offs + PH_SWEEP * (bv.njobs + 1);
  const int jb = batch_job(offs, bv.njobs, (int)blockIdx.x);
  const JobDesc& J = bv.jobs[jb];
  const FluxOut<T> out = flux_out<T>(global_ptr((unsigned char*)J.F), J.d.sv);
  const SweepArgs<T> a{global_ptr(corrector ? J.Ph : J.P), global_ptr(FaceTables<T>::f1(J.t)),
                       global_ptr(FaceTables<T>::f2(J.t)), global_ptr(FaceTables<T>::f3(J.t)), out,
                       J.E ? out.m : nullptr, J.up.idx1, J.up.idx2, J.up.idx3, (T)J.p.gam, J.up.polar_lo,
                       J.up.polar_hi};
  const Dims d = J.d;  // kept: read from the table where needed, the FP64 MC predictor spills 6 registers
  sweep_body<RECON, T, GEO, CTOP, BX, BY>(d, a, (int)blockIdx.x - offs[jb], CTOP ? global_ptr(J.ctr->ctop) : nullptr);
}

template <int RECON, typename T, int BX, int BY>
constexpr size_t tile_bytes() {
  return ((size_t)NV * PlaneShape<RECON, BX, BY>::PLANE + (size_t)NEXCH * BX * BY) * sizeof(T);
}

// A kernel may use more dynamic LDS than the default 64 KiB only once the limit
// is raised for it, on each device: the default FP64 MC pass takes 75 KB.
template <auto KERNEL>
hipError_t allow_lds(size_t bytes) {
  constexpr int DEVICES = 64;
  static std::atomic<bool> raised[DEVICES];
  if (bytes <= 65536) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || (dev < DEVICES && raised[dev].load())) return e;
  e = hipFuncSetAttribute((const void*)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && dev < DEVICES) raised[dev].store(true);
  return e;
}

// f(std::integral_constant BX, BY) for a block shape
template <int RECON, typename T, int SHAPE, typename F>
hipError_t with_extents(F f) {
  constexpr bool MIXED = std::is_same<T, float>::value;
  return f(std::integral_constant<int, sweep_bx(SHAPE, RECON, MIXED)>(),
           std::integral_constant<int, sweep_by(SHAPE, RECON, MIXED)>());
}
template <int RECON, typename T, typename F>
hipError_t with_shape(int shape, F f) {
  if (shape == SWEEP_NARROW) return with_extents<RECON, T, SWEEP_NARROW>(f);
  if (shape == SWEEP_SMALL) return with_extents<RECON, T, SWEEP_SMALL>(f);
  return with_extents<RECON, T, SWEEP_LARGE>(f);
}

template <int RECON, typename T, int GEO, bool CTOP>
hipError_t launch_ctop(const Dims& d, const SweepArgs<T>& a, unsigned long long* ctop, hipStream_t s) {
  return with_shape<RECON, T>(d.shape, [&](auto bx, auto by) {
    constexpr int BX = decltype(bx)::value, BY = decltype(by)::value;
    constexpr size_t lds = tile_bytes<RECON, T, BX, BY>();
    const hipError_t e = allow_lds<sweep_kernel<RECON, T, GEO, CTOP, BX, BY>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((sweep_kernel<RECON, T, GEO, CTOP, BX, BY>), dim3(sweep_blocks(d)), dim3(BX, BY, 1), lds, s, d, a,
                       ctop);
    return hipGetLastError();
  });
}

template <int RECON, typename T, int GEO>
hipError_t launch_speeds(const Dims& d, const SweepArgs<T>& a, unsigned long long* ctop, hipStream_t s) {
  return with_shape<RECON, T>(d.shape, [&](auto bx, auto by) {
    constexpr int BX = decltype(bx)::value, BY = decltype(by)::value;
    constexpr size_t lds = (size_t)NV * (PlaneShape<RECON, BX, BY>::PLANE + BX) * sizeof(T);
    const hipError_t e = allow_lds<speed_kernel<RECON, T, GEO, BX, BY>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((speed_kernel<RECON, T, GEO, BX, BY>), dim3(sweep_blocks(d)), dim3(BX, BY, 1), lds, s, d, a, ctop);
    return hipGetLastError();
  });
}

template <int RECON, typename T, int GEO>
hipError_t launch_geo(const Dims& d, const Tables& t, const UpdateParams& up, const double* P, void* F,
                      bool mass, unsigned long long* ctop, hipStream_t s) {
  const FluxOut<T> out = flux_out<T>((unsigned char*)F, d.sv);
  const SweepArgs<T> a{P,       FaceTables<T>::f1(t), FaceTables<T>::f2(t), FaceTables<T>::f3(t), out, mass ? out.m : nullptr,
                       up.idx1, up.idx2,              up.idx3,              (T)up.gam,            up.polar_lo, up.polar_hi};
  if (!F) return launch_speeds<RECON, T, GEO>(d, a, ctop, s);
  if (ctop) return launch_ctop<RECON, T, GEO, true>(d, a, ctop, s);
  return launch_ctop<RECON, T, GEO, false>(d, a, ctop, s);
}

// Cartesian Kerr-Schild in FP64 computes its face geometry instead of
// streaming the 3D face tables (most of the bytes the pass moved); the
// FP32 pass reads the float tables, cheaper than evaluating the metric in
// FP64; the other coordinates read their 2D tables
template <int RECON, typename T>
hipError_t launch_for(const grmhd_problem& p, const Dims& d, const Tables& t, const UpdateParams& up, const double* P,
                      void* F, bool mass, unsigned long long* ctop, hipStream_t s) {
  if (p.coords != GRMHD_KERR_CKS) return launch_geo<RECON, T, GEO_AXI>(d, t, up, P, F, mass, ctop, s);
  if constexpr (std::is_same<T, double>::value)
    return launch_geo<RECON, T, GEO_CKS>(d, t, up, P, F, mass, ctop, s);
  else return launch_geo<RECON, T, GEO_TABLE>(d, t, up, P, F, mass, ctop, s);
}

// a batch whose jobs all have g_23 = beta^3 = 0 reads the shorter tables (the
// same bits: the components left out are zeros)
template <int RECON, typename T, int GEO, bool CTOP>
hipError_t launch_batch_ctop(const BatchView& bv, dim3 grd, int c, hipStream_t s) {
  return with_shape<RECON, T>(bv.shape, [&](auto bx, auto by) {
    constexpr int BX = decltype(bx)::value, BY = decltype(by)::value;
    constexpr size_t lds = tile_bytes<RECON, T, BX, BY>();
    const hipError_t e = allow_lds<sweep_batch_kernel<RECON, T, GEO, CTOP, BX, BY>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((sweep_batch_kernel<RECON, T, GEO, CTOP, BX, BY>), grd, dim3(BX, BY, 1), lds, s, bv, c);
    return hipGetLastError();
  });
}

template <int RECON, typename T>
hipError_t launch_batch_for(const BatchView& bv, dim3 grd, int c, bool ctop, hipStream_t s) {
  if (bv.axi)
    return ctop ? launch_batch_ctop<RECON, T, GEO_AXI, true>(bv, grd, c, s)
                : launch_batch_ctop<RECON, T, GEO_AXI, false>(bv, grd, c, s);
  return ctop ? launch_batch_ctop<RECON, T, GEO_TABLE, true>(bv, grd, c, s)
              : launch_batch_ctop<RECON, T, GEO_TABLE, false>(bv, grd, c, s);
}

}  // namespace

unsigned sweep_blocks(const Dims& d) { return (unsigned)sweep_grid(d, d.sbx, d.sby); }

hipError_t launch_sweeps(const grmhd_problem& p, bool mixed, const Dims& d, const Tables& t, const UpdateParams& up,
                         const double* P, void* F, bool mass, unsigned long long* ctop, hipStream_t s) {
  if (mixed) {
    if (p.recon == GRMHD_RECON_MC) return launch_for<GRMHD_RECON_MC, float>(p, d, t, up, P, F, mass, ctop, s);
    return launch_for<GRMHD_RECON_WENO5, float>(p, d, t, up, P, F, mass, ctop, s);
  }
  if (p.recon == GRMHD_RECON_MC) return launch_for<GRMHD_RECON_MC, double>(p, d, t, up, P, F, mass, ctop, s);
  return launch_for<GRMHD_RECON_WENO5, double>(p, d, t, up, P, F, mass, ctop, s);
}

hipError_t launch_batch_sweeps(const BatchView& bv, const int* totals, int recon, bool mixed, bool corrector,
                               bool want_ctop, hipStream_t s) {
  const dim3 grd(totals[PH_SWEEP]);
  const int c = corrector ? 1 : 0;
  const bool w = want_ctop;
  if (mixed) {
    if (recon == GRMHD_RECON_MC) return launch_batch_for<GRMHD_RECON_MC, float>(bv, grd, c, w, s);
    return launch_batch_for<GRMHD_RECON_WENO5, float>(bv, grd, c, w, s);
  }
  if (recon == GRMHD_RECON_MC) return launch_batch_for<GRMHD_RECON_MC, double>(bv, grd, c, w, s);
  return launch_batch_for<GRMHD_RECON_WENO5, double>(bv, grd, c, w, s);
}
