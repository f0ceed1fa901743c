// Explicit instances of the large kernels.  Each group is compiled in a
// translation unit of its own (inst_*.hip), so the library builds in parallel;
// every other unit sees the `extern` declarations below.  X: `extern` or
// nothing; Geo: KS, Flat or Dense.
#pragma once
#include "adjoint.h"

#define INST_FLUX(X, Geo)                                                                         \
  X template __global__ void k_flux_all<Geo, double>(Ctx, FluxSegs, const double*, const          \
      double*, const double*, double*, double*, const double*);                                   \
  X template __global__ void k_flux_all_s<Geo, double>(Ctx, FluxSegs, const double*, const        \
      double*, const double*, double*, double*, const double*, double*);

#define INST_FLUX_STAG(X, Geo)                                                                    \
  X template __global__ void k_flux_all_stag<Geo, double, false>(Ctx, FluxSegs, const             \
      double*, const double*, const double*, double*, double*, const double*, double*, const      \
      double*, double*, double*);                                                                 \
  X template __global__ void k_flux_all_stag<Geo, double, true>(Ctx, FluxSegs, const              \
      double*, const double*, const double*, double*, double*, const double*, double*, const      \
      double*, double*, double*);

#define INST_FLUX_F32(X, Geo)                                                                     \
  X template __global__ void k_flux_all<Geo, float>(Ctx, FluxSegs, const double*, const           \
      double*, const double*, double*, double*, const double*);                                   \
  X template __global__ void k_flux_all_s<Geo, float>(Ctx, FluxSegs, const double*, const         \
      double*, const double*, double*, double*, const double*, double*);                          \
  X template __global__ void k_flux_all_stag<Geo, float, false>(Ctx, FluxSegs, const              \
      double*, const double*, const double*, double*, double*, const double*, double*, const      \
      double*, double*, double*);                                                                 \
  X template __global__ void k_flux_all_stag<Geo, float, true>(Ctx, FluxSegs, const double*,      \
      const double*, const double*, double*, double*, const double*, double*, const double*,      \
      double*, double*);

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
INST_FLUX(extern, KS)
INST_FLUX(extern, Flat)
INST_FLUX(extern, Dense)
#endif
#ifndef INST_HERE_FLUX_STAG
INST_FLUX_STAG(extern, KS)
INST_FLUX_STAG(extern, Flat)
#endif
#ifndef INST_HERE_FLUX_F32
INST_FLUX_F32(extern, Dense)
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
