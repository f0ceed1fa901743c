// Face fluxes of the FP64 step.
#define INST_HERE_FLUX
#define INST_HERE_FLUX_STAG
#include "instances.h"

INST_FLUX(, KS)
INST_FLUX(, Flat)
INST_FLUX_STAG(, KS)
INST_FLUX_STAG(, Flat)
