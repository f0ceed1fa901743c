// Host build of the device solver headers: the URAD attempt as a batch's
// cascade runs it, an evaluation's gas inversion taken a few Newton steps at a
// time, its bisection apart from them and the root handed to the evaluation
// (the stages of k_cascade_urad), the result through the cell's record as
// k_cascade_finish reads it.  It must give the bits of implicit_cell resuming
// from the same first attempt.  Arguments: batch file, steps a trip.  Prints
// one line: "cells <n> differing <n> parts <n> bisected <n> rootless <n>".
#define DEV __host__ __device__ inline
#include <hip/hip_runtime.h>
#include <cmath>
__host__ inline bool isfinite(double x) { return std::isfinite(x); }
#include "../../paper_1312_6127_amd/csrc/kernels.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

static bool same_bits(const CellOut& a, const CellOut& b) {
  return a.status == b.status && a.iters == b.iters && std::memcmp(&a.err, &b.err, 8) == 0 &&
         std::memcmp(a.P, b.P, sizeof(a.P)) == 0 && std::memcmp(a.U, b.U, sizeof(a.U)) == 0;
}

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  const int steps = atoi(argv[2]);
  FILE* f = fopen(argv[1], "rb");
  if (!f) return 2;
  long n;
  double prm[10];
  if (fread(&n, 8, 1, f) != 1 || fread(prm, 8, 10, f) != 10) return 2;
  std::vector<double> Ui(12 * n), Pg(12 * n), dt(n), ca(n), ce(n);
  size_t got = fread(Ui.data(), 8, 12 * n, f) + fread(Pg.data(), 8, 12 * n, f) +
               fread(dt.data(), 8, n, f) + fread(ca.data(), 8, n, f) + fread(ce.data(), 8, n, f);
  fclose(f);
  if (got != (size_t)(27 * n)) return 2;
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
  Metric m;
  flat_metric(m);
  long cells = 0, diff = 0, parts = 0, bisected = 0, rootless = 0;
  for (long cc = 0; cc < n; cc++) {
    double u[12], p[12];
    for (int q = 0; q < 12; q++) {
      u[q] = Ui[q * n + cc];
      p[q] = Pg[q * n + cc];
    }
    CellOut ref, out;
    Best b;
    int it = 0, tr = 0;
    bool ext = false;
    if (implicit_fast(m, ph, o, u, p, dt[cc], ca[cc], ce[cc], out, b, it, ext, tr) || ext) continue;
    cells++;
    double rd[14];
    int ri[2];
    RecBuf R;
    R.d = rd;
    R.i = ri;
    R.cap = 1;
    rec_store(R, 0, b, it, out.status);
    implicit_cell(m, ph, o, u, p, dt[cc], ca[cc], ce[cc], ref, &R, 0, false);
    // the lane of k_cascade_urad
    Cell c;
    cell_setup(m, u, dt[cc], ca[cc], ce[cc], c);
    UradLane L;
    Best b0;
    int it0;
    rec_load(R, 0, b0, it0);
    const double* src = (b0.ok && b0.eT < 1e-4) ? b0.P : p;
    rad_cons4(m, src, L.p);
    for (int q = 0; q < 5; q++) L.Pn[q] = src[q];
    L.iters = it0;
    L.mode = UM_START;
    MhdIter in;
    int stage = UE_NONE;
    for (long guard = 0; guard < 100000; guard++) {
      bool ended = false;
      if (stage == UE_NONE) {
        ended = urad_before(c, o, L);
        if (!ended) {
          const MhdC gc = urad_gas(c, ph, L.p);
          stage = mhd_start(m, gc, L.Pn[1], L.Pn + 2, in) ? UE_NEWTON : UE_FAILED;
        }
      }
      if (stage == UE_NEWTON) {
        const MhdC gc = urad_gas(c, ph, L.p);
        if (mhd_iterate<false>(gc, in, steps)) stage = in.ok ? UE_ROOT : UE_BISECT;
        else parts++;
      } else if (stage == UE_BISECT) {   // a trip later, as where lanes wait
        const MhdC gc = urad_gas(c, ph, L.p);
        stage = mhd_bisect(gc, in.Wp) ? UE_FAILED : UE_ROOT;
        bisected++;
      }
      if (stage == UE_ROOT || stage == UE_FAILED) {
        Eval ev;
        double Jn[4][4];
        if (stage == UE_ROOT) {
          eval_urad_jac(c, ph, L.p, L.Pn, ev, Jn, &in.Wp);
        } else {
          ev.ok = 0;
          ev.eT = INFINITY;
          rootless++;
        }
        ended = urad_after(ev, Jn, L);
        stage = UE_NONE;
      }
      if (ended) break;
    }
    rec_urad(R, 0, L.best, L.iters);
    // k_cascade_finish
    Best best;
    int its;
    rec_load(R, 0, best, its, c.B);
    const int st = R.i[0] >> REC_STATUS, bm = best.ok ? best.ok >> 1 : -1;
    if (bm < 0) failed_out(u, p, st, its, out);
    else finalize(c, ph, o, best, bm, st, its, u, out);
    if (!same_bits(out, ref)) diff++;
  }
  printf("cells %ld differing %ld parts %ld bisected %ld rootless %ld\n", cells, diff, parts, bisected,
         rootless);
  return 0;
}
