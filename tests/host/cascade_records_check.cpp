// Host build of the device solver headers: a cell's full cascade resumed from
// the record of its PMHD and URAD attempts, as a batch's kernels leave and
// take it, must give the bits of the same cascade from scratch.  Prints one
// line: "resumed <n> urad <n> differing <n>" (urad: outputs whose solution is
// the URAD attempt's, its conserved radiation taken from the record).
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
  long resumed = 0, urad = 0, diff = 0;
  for (long cc = 0; cc < n; cc++) {
    double u[12], p[12];
    for (int q = 0; q < 12; q++) {
      u[q] = Ui[q * n + cc];
      p[q] = Pg[q * n + cc];
    }
    CellOut out;
    Best b;
    int it = 0, tr = 0;
    bool ext = false;
    if (implicit_fast(m, ph, o, u, p, dt[cc], ca[cc], ce[cc], out, b, it, ext, tr) || ext) continue;
    double rd[14];
    int ri[2];
    RecBuf R;
    R.d = rd;
    R.i = ri;
    R.cap = 1;
    rec_store(R, 0, b, it, out.status);
    // the URAD attempt
    Cell c;
    cell_setup(m, u, dt[cc], ca[cc], ce[cc], c);
    const double* src = (b.ok && b.eT < 1e-4) ? b.P : p;
    double x0[4], P0[5];
    rad_cons4(m, src, x0);
    for (int q = 0; q < 5; q++) P0[q] = src[q];
    Best bu;
    bu.eT = INFINITY;
    bu.ok = 0;
    newton<M_URAD>(c, ph, o, x0, P0, bu, it);
    rec_urad(R, 0, bu, it);
    const double Si = entropy_cons(ph.gam, m, p);
    CellOut ref;
    implicit_cell_full(m, ph, o, u, Si, p, dt[cc], ca[cc], ce[cc], ref);
    implicit_cell_full(m, ph, o, u, Si, p, dt[cc], ca[cc], ce[cc], out, &R, 0, 2);
    resumed++;
    urad += (out.status & (GRRMHD_ST_URAD | GRRMHD_ST_ENTROPY | GRRMHD_ST_STAGED)) == GRRMHD_ST_URAD;
    if (!same_bits(out, ref)) diff++;
  }
  printf("resumed %ld urad %ld differing %ld\n", resumed, urad, diff);
  return 0;
}
