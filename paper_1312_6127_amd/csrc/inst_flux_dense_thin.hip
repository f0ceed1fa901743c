// The dense form's face fluxes on grids of thin planes.
#define INST_HERE_FLUX_DENSE_THIN
#include "instances.h"

INST_FLUX_DENSE(, true)
