// Explicit instances of the large kernels.  Each group is compiled in a
// translation unit of its own (inst_*.hip), so the library builds in parallel;
// every other unit sees the `extern` declarations below.  X: `extern` or
// nothing; Geo: KS, Flat or Dense.
#pragma once
#include "adjoint.h"

#define INST_FLUX(X, Geo, T, Thin)                                                                \
  X template __global__ void k_flux_all<Geo, T, Thin>(Ctx, FluxSegs, const double*, const         \
      double*, const double*, double*, double*, const double*);                                   \
  X template __global__ void k_flux_all_s<Geo, T, Thin>(Ctx, FluxSegs, const double*, const       \
      double*, const double*, double*, double*, const double*, double*);

#define INST_FLUX_STAG(X, Geo, T, Thin)                                                           \
  X template __global__ void k_flux_all_stag<Geo, T, false, Thin>(Ctx, FluxSegs, const            \
      double*, const double*, const double*, double*, double*, const double*, double*, const      \
      double*, double*, double*);                                                                 \
  X template __global__ void k_flux_all_stag<Geo, T, true, Thin>(Ctx, FluxSegs, const             \
      double*, const double*, const double*, double*, double*, const double*, double*, const      \
      double*, double*, double*);

// the FP64 step's faces; those of the dense form (FP64 and FP32)
#define INST_FLUX_STEP(X, Thin)                                                                   \
  INST_FLUX(X, KS, double, Thin)                                                                  \
  INST_FLUX(X, Flat, double, Thin)                                                                \
  INST_FLUX_STAG(X, KS, double, Thin)                                                             \
  INST_FLUX_STAG(X, Flat, double, Thin)
#define INST_FLUX_DENSE(X, Thin)                                                                  \
  INST_FLUX(X, Dense, double, Thin)                                                               \
  INST_FLUX(X, Dense, float, Thin)                                                                \
  INST_FLUX_STAG(X, Dense, float, Thin)

#define INST_IMPLICIT(X, Geo)                                                                     \
  X template __global__ void k_implicit<Geo>(Ctx, int, const double*, const double*, double,      \
      const double*, const double*, const double*, double*, double*, int*, int*, double*,         \
      Work, const int*, int*);                                                                    \
  X template __global__ void k_implicit_list<Geo, false>(Ctx, const double*, const double*,       \
      double, const double*, const double*, const double*, double*, double*, int*, int*,          \
      double*, Work, const double*);

#define INST_CASCADE(X, Geo)                                                                      \
  X template __global__ void k_implicit_list<Geo, true>(Ctx, const double*, const double*,        \
      double, const double*, const double*, const double*, double*, double*, int*, int*,          \
      double*, Work, const double*);

#define INST_BATCH(X, Geo)                                                                        \
  X template __global__ void k_implicit_batch<Geo>(Ctx, long, const double*, const double*,       \
      const double*, const double*, const double*, double*, double*, int*, int*, double*,         \
      Work);                                                                                      \
  X template __global__ void k_cold_batch_list<Geo>(Ctx, long, const double*, const double*,      \
      const double*, const double*, const double*, double*, double*, int*, int*, double*,         \
      Work);                                                                                      \
  X template __global__ void k_cascade_urad<Geo>(Ctx, long, const double*, const double*,         \
      const double*, const double*, const double*, double*, double*, int*, int*, double*,         \
      Work, int*, Work);                                                                          \
  X template __global__ void k_cascade_finish<Geo>(Ctx, long, const double*, const double*,       \
      const double*, const double*, const double*, double*, double*, int*, int*, double*,         \
      Work, Work);                                                                                \
  X template __global__ void k_implicit_persist<Geo>(Ctx, long, const double*, const              \
      double*, const double*, const double*, const double*, double*, double*, int*, int*,         \
      double*, int*, Work);                                                                       \
  X template __global__ void k_iter_start<Geo>(Ctx, long, const double*, const double*,           \
      const double*, const double*, const double*, double*, int*, int*, int*, Work);              \
  X template __global__ void k_iter_step<Geo>(Ctx, long, const double*, const double*, const      \
      double*, const double*, double*, int*, const int*, const int*, int*, int*, double*,         \
      double*, int*, int*, double*, Work);

#define INST_BATCH_REST(X, Geo)                                                                   \
  X template __global__ void k_implicit_batch_list<Geo>(Ctx, long, const double*, const           \
      double*, const double*, const double*, const double*, double*, double*, int*, int*,         \
      double*, Work);                                                                             \
  X template __global__ void k_rest_batch_list<Geo>(Ctx, long, const double*, const double*,      \
      const double*, const double*, const double*, double*, double*, int*, int*, double*,         \
      Work, Work);

#define INST_ADJ_FLUX(X, Geo)                                                                     \
  X template __global__ void k_adj_flux<Geo, false>(Ctx, AdjFaces, double, const double*, const   \
      double*, const double*, const double*, const double*, const double*, double*, long,         \
      double*, const double*, double*, const double*);                                            \
  X template __global__ void k_adj_flux<Geo, true>(Ctx, AdjFaces, double, const double*, const    \
      double*, const double*, const double*, const double*, const double*, double*, long,         \
      double*, const double*, double*, const double*);

#define INST_ADJ_IMPLICIT(X, Geo)                                                                 \
  X template __global__ void k_adj_implicit<Geo, false>(Ctx, double, const double*, const         \
      double*, const double*, const int*, const double*, const double*, const double*, const      \
      double*, double*, double*, const double*, double*);                                         \
  X template __global__ void k_adj_implicit<Geo, true>(Ctx, double, const double*, const          \
      double*, const double*, const int*, const double*, const double*, const double*, const      \
      double*, double*, double*, const double*, double*);

#ifndef INST_HERE_FLUX
INST_FLUX_STEP(extern, false)
#endif
#ifndef INST_HERE_FLUX_THIN
INST_FLUX_STEP(extern, true)
#endif
#ifndef INST_HERE_FLUX_DENSE
INST_FLUX_DENSE(extern, false)
#endif
#ifndef INST_HERE_FLUX_DENSE_THIN
INST_FLUX_DENSE(extern, true)
#endif
#ifndef INST_HERE_IMPLICIT
INST_IMPLICIT(extern, KS)
INST_IMPLICIT(extern, Flat)
INST_IMPLICIT(extern, Dense)
#endif
#ifndef INST_HERE_CASCADE
INST_CASCADE(extern, Dense)
#endif
#ifndef INST_HERE_BATCH
INST_BATCH(extern, Dense)
#endif
#ifndef INST_HERE_BATCH_REST
INST_BATCH_REST(extern, Dense)
#endif
#ifndef INST_HERE_ADJ_FLUX
INST_ADJ_FLUX(extern, Dense)
#endif
#ifndef INST_HERE_ADJ_IMPLICIT
INST_ADJ_IMPLICIT(extern, Dense)
#endif
