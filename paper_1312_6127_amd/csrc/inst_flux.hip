// Face fluxes of the FP64 step.
#define INST_HERE_FLUX
#include "instances.h"

INST_FLUX_STEP(, false)
