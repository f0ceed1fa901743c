// Face fluxes of the FP64 step on grids of thin planes.
#define INST_HERE_FLUX_THIN
#include "instances.h"

INST_FLUX_STEP(, true)
