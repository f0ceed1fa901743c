// Host build of the device solver headers: Kerr-Schild cells within rounding
// of the extreme regime's threshold.  The first kernel's closed form decides
// the regime; the rest of the cascade must follow it, whatever an earlier
// launch left in the cell's record and whatever its own form of the same
// expression would say.  Prints one line: "cells <n> extreme <n> split <n>
// differing <n>" (split: cells that the two forms decide differently).
#define DEV __host__ __device__ inline
#include <hip/hip_runtime.h>
#include <cmath>
__host__ inline bool isfinite(double x) { return std::isfinite(x); }
#include "../../paper_1312_6127_amd/csrc/kernels.h"
#include <cstdio>
#include <cstring>
#include <vector>

static bool same_bits(const CellOut& a, const CellOut& b) {
  return a.status == b.status && a.iters == b.iters && std::memcmp(&a.err, &b.err, 8) == 0 &&
         std::memcmp(a.P, b.P, sizeof(a.P)) == 0 && std::memcmp(a.U, b.U, sizeof(a.U)) == 0;
}

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  FILE* f = fopen(argv[1], "rb");
  if (!f) return 2;
  long n;
  double prm[9];
  if (fread(&n, 8, 1, f) != 1 || fread(prm, 8, 9, f) != 9) return 2;
  // per cell: the metric's table entries, U_(i), P_n, dt
  const int W = GE_NFACE + 25;
  std::vector<double> cells(W * n);
  if (fread(cells.data(), 8, W * n, f) != (size_t)(W * n)) return 2;
  fclose(f);
  Phys ph;
  ph.gam = prm[0];
  ph.arad = prm[1];
  ph.gamma_max = prm[2];
  const double G = prm[2] * prm[2];
  ph.ymax = 16.0 * G * (G - 1.0) / ((4.0 * G - 1.0) * (4.0 * G - 1.0));
  Opts o;
  o.tol_pmhd = prm[3];
  o.tol_urad = prm[4];
  o.tol_accept = prm[5];
  o.tol_fail = prm[6];
  o.max_iter = (int)prm[7];
  o.roundoff = (int)prm[8];
  long listed = 0, next = 0, split = 0, diff = 0;
  for (long cc = 0; cc < n; cc++) {
    const double* d = &cells[W * cc];
    const double *u = d + GE_NFACE, *p = u + 12, dt = p[12], ca = 1.0, ce = 1.0;
    KSMetric<double> m;
    m.load(d, 1, 0);
    CellOut out[3];
    Best b;
    int it = 0, tr = 0;
    bool ext = false;
    if (implicit_first(m, ph, o, u, p, dt, ca, ce, out[0], b, it, ext, tr)) continue;
    listed++;
    next += ext;
    CellT<KSMetric<double>> c;
    Prep pr;
    prepare(m, ph, u, p, dt, ca, ce, c, pr);
    split += pr.extreme != ext;
    bool ok = true;
    for (int full = 0; full < 2; full++) {
      for (int k = 0; k < 2; k++) {
        // what an earlier launch left in the slot: another cell's solution
        Best old;
        for (int q = 0; q < 12; q++) old.P[q] = p[q] * (1.0 + 0.1 * k);
        old.eT = k ? 1e-16 : 1e-5;
        old.radflags = 0;
        old.ok = 1;
        double rd[13];
        int ri[2];
        RecBuf R;
        R.d = rd;
        R.i = ri;
        R.cap = 1;
        rec_store(R, 0, old, 7);
        rec_first(R, 0, ext, b, it);
        if (full)
          implicit_cell_full(m, ph, o, u, entropy_cons(ph.gam, m, p), p, dt, ca, ce, out[k], &R, 0, 1);
        else
          implicit_cell(m, ph, o, u, p, dt, ca, ce, out[k], &R, 0);
        ok = ok && ((out[k].status & GRRMHD_ST_EXTREME) != 0) == ext;
      }
      ok = ok && same_bits(out[0], out[1]);
    }
    if (!ok) diff++;
  }
  printf("cells %ld extreme %ld split %ld differing %ld\n", listed, next, split, diff);
  return 0;
}
