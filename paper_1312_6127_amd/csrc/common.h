// Internal definitions shared by the HIP kernels and the host side of the
// library: the kernel context passed by value to every launch, geometry
// table layout, and index helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/grrmhd.h"
#include "dual.h"

#ifndef DEV
#define DEV __device__ __forceinline__
#endif

// Geometry tables: 2-D (x1, x2) arrays broadcast over x3, because both
// metrics are independent of x3 (phi).  Field-major [field][j][i].
// Symmetric 4x4 tensors store the 10 components (00,01,02,03,11,12,13,22,23,33).
enum {
  GE_GCOV = 0,     // 10
  GE_GCON = 10,    // 10
  GE_GDET = 20,
  GE_ALPHA = 21,
  GE_NFACE = 22,   // fields stored at faces
  GE_DG1 = 22,     // d g_{mn}/dx1, 10 (cell centres only)
  GE_DG2 = 32,     // d g_{mn}/dx2, 10
  GE_NCENTER = 42
};

DEV constexpr int sym(int a, int b) {
  return (a <= b) ? (a == 0 ? b : (a == 1 ? 3 + b : (a == 2 ? 5 + b : 9)))
                  : (b == 0 ? a : (b == 1 ? 3 + a : (b == 2 ? 5 + a : 9)));
}

struct Ctx {
  int n[3], ng[3], N[3];
  long Ntot;
  long st[3];          // strides of i, j, k
  int npos;            // N1 * N2 (geometry table stride)
  double dx[3], xlo[3];
  int metric;
  int bc_lo[3], bc_hi[3];
  double gam, arad, gamma_max, ymax, courant;
  int flux;
  int recon;           // GRRMHD_RECON_MC or GRRMHD_RECON_PPM
  int cold;            // cold MHD limit for cells with no energy solution
  int cascade;         // 1: the full method cascade (PRAD, staged, entropy)
  int ct;              // 0: flux-CT on the cell-centred field; 1: staggered face field
  int mixed_i;         // FP32-mixed: cells with x1 index >= mixed_i take the FP32 face path
  double tol_pmhd, tol_urad, tol_accept, tol_fail;
  int max_iter, roundoff;
  double rho_floor, u_floor, bsq_rho_max, bsq_u_max, u_rho_max, erad_floor;
  const double* geo_c;   // [GE_NCENTER][npos]
  const double* geo_f1;  // [GE_NFACE][npos] at x1 faces
  const double* geo_f2;  // [GE_NFACE][npos] at x2 faces
};

// Real type of the literals and metric coefficients that go with a scalar
// T: float on the FP32 face path, double otherwise (double and Dual<N>).
template <class T>
struct RealOf {
  using type = double;
};
template <>
struct RealOf<float> {
  using type = float;
};

// Metric at one point.  lo, up: g_ab, g^ab; gam(i, j): the normal observer's
// spatial inverse metric g^{ij} - g^{ti} g^{tj}/g^{tt}; zlo, zup, zgam: known
// at compile time to vanish.  Three forms, and a kernel is compiled for the
// ones it needs:
//   DenseMetric  every component, for either space-time.  The adjoint, the
//                FP32 face path and the batched solve: their results amplify
//                the last bit of an intermediate (the 96x48x24 disk's gradient
//                moves by 1e-6 when its input moves by one ulp; a batch's
//                iteration counts and failed cells move likewise), so they
//                keep one order of operations;
//   KSMetric     Kerr-Schild without the components that vanish there;
//   FlatMetric   Minkowski.
// The FP64 step runs on the last two: products with a vanishing component are
// never formed (a contraction keeps 10 of its 16 terms on Kerr-Schild, 4 in
// flat space) and a point takes 16 registers or none instead of 22.
template <class R>
struct DenseMetric {
  static constexpr bool dense = true, diagonal = false;
  R gcov[10], gcon[10], gdet, alpha;
  DEV static constexpr bool zlo(int, int) { return false; }
  DEV static constexpr bool zup(int, int) { return false; }
  DEV static constexpr bool zgam(int, int) { return false; }
  DEV R lo(int a, int b) const { return gcov[sym(a, b)]; }
  DEV R up(int a, int b) const { return gcon[sym(a, b)]; }
  DEV R gam(int i, int j) const { return up(i + 1, j + 1) - up(0, i + 1) * up(0, j + 1) / up(0, 0); }
  DEV void load(const double* tab, int npos, int pos) {
#pragma unroll
    for (int q = 0; q < 10; q++) gcov[q] = (R)tab[(GE_GCOV + q) * npos + pos];
#pragma unroll
    for (int q = 0; q < 10; q++) gcon[q] = (R)tab[(GE_GCON + q) * npos + pos];
    gdet = (R)tab[GE_GDET * npos + pos];
    alpha = (R)tab[GE_ALPHA * npos + pos];
  }
};

template <class R>
struct FlatMetric {
  static constexpr bool dense = false, diagonal = true;
  static constexpr R gdet = R(1.0), alpha = R(1.0);
  DEV static constexpr bool zlo(int a, int b) { return a != b; }
  DEV static constexpr bool zup(int a, int b) { return a != b; }
  DEV static constexpr bool zgam(int i, int j) { return i != j; }
  DEV static constexpr R lo(int a, int b) { return a != b ? R(0.0) : (a == 0 ? R(-1.0) : R(1.0)); }
  DEV static constexpr R up(int a, int b) { return lo(a, b); }
  DEV static constexpr R gam(int i, int j) { return lo(i + 1, j + 1); }
  DEV void load(const double*, int, int) {}
};

template <class R>
struct KSMetric {
  static constexpr bool dense = false, diagonal = false;
  R g00, g01, g03, g11, g13, g22, g33;
  R u00, u01, u11, u13, u22, u33;
  R gdet, alpha;
  R gam11;
  // tt, tr, t phi, rr, r phi, theta theta, phi phi; inverse: no t phi
  DEV static constexpr bool zlo(int a, int b) { return (a == 2) != (b == 2); }
  DEV static constexpr bool zup(int a, int b) { return zlo(a, b) || (a + b == 3 && a * b == 0); }
  DEV static constexpr bool zgam(int i, int j) { return zlo(i + 1, j + 1); }
  DEV R lo(int a, int b) const {
    const int s = sym(a, b);
    return s == 0 ? g00 : s == 1 ? g01 : s == 3 ? g03 : s == 4 ? g11 : s == 6 ? g13
           : s == 7 ? g22 : s == 9 ? g33 : R(0.0);
  }
  DEV R up(int a, int b) const {
    const int s = sym(a, b);
    return s == 0 ? u00 : s == 1 ? u01 : s == 4 ? u11 : s == 6 ? u13 : s == 7 ? u22
           : s == 9 ? u33 : R(0.0);
  }
  // g^{t theta} = g^{t phi} = 0: only the rr component differs from g^{ij}
  DEV R gam(int i, int j) const { return (i == 0 && j == 0) ? gam11 : up(i + 1, j + 1); }
  DEV void load(const double* tab, int npos, int pos) {
    auto at = [&](int f) { return (R)tab[f * npos + pos]; };
    g00 = at(GE_GCOV + sym(0, 0));
    g01 = at(GE_GCOV + sym(0, 1));
    g03 = at(GE_GCOV + sym(0, 3));
    g11 = at(GE_GCOV + sym(1, 1));
    g13 = at(GE_GCOV + sym(1, 3));
    g22 = at(GE_GCOV + sym(2, 2));
    g33 = at(GE_GCOV + sym(3, 3));
    u00 = at(GE_GCON + sym(0, 0));
    u01 = at(GE_GCON + sym(0, 1));
    u11 = at(GE_GCON + sym(1, 1));
    u13 = at(GE_GCON + sym(1, 3));
    u22 = at(GE_GCON + sym(2, 2));
    u33 = at(GE_GCON + sym(3, 3));
    gdet = at(GE_GDET);
    alpha = at(GE_ALPHA);
    gam11 = u11 - u01 * u01 / u00;
  }
};

// What a kernel is compiled for.
struct KS {
  static constexpr bool closed = true, closed_faces = true;
  DEV static constexpr bool curved(const Ctx&) { return true; }
  template <class R>
  using M = KSMetric<R>;
};
struct Flat {
  // Faces keep face_state's order of operations: 200 steps of a shock tube
  // amplify a face's last bit to 1e-10 of a field, and its 9 us launches are
  // latency, not arithmetic
  static constexpr bool closed = true, closed_faces = false;
  DEV static constexpr bool curved(const Ctx&) { return false; }
  template <class R>
  using M = FlatMetric<R>;
};
struct Dense {
  static constexpr bool closed = false, closed_faces = false;   // no closed forms
  DEV static bool curved(const Ctx& C) { return C.metric == GRRMHD_KERR_SCHILD; }
  template <class R>
  using M = DenseMetric<R>;
};

using Metric = DenseMetric<double>;

template <class M>
DEV void load_metric(const double* tab, int npos, int pos, M& m) {
  m.load(tab, npos, pos);
}

DEV void flat_metric(FlatMetric<double>&) {}
DEV void flat_metric(Metric& m) {
#pragma unroll
  for (int q = 0; q < 10; q++) m.gcov[q] = m.gcon[q] = 0.0;
  m.gcov[0] = m.gcon[0] = -1.0;
  m.gcov[4] = m.gcon[4] = 1.0;
  m.gcov[7] = m.gcon[7] = 1.0;
  m.gcov[9] = m.gcon[9] = 1.0;
  m.gdet = 1.0;
  m.alpha = 1.0;
}
