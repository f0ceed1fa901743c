// Face fluxes in the dense form: FP32, and FP64 for the Courant step and the adjoint.
#define INST_HERE_FLUX_DENSE
#include "instances.h"

INST_FLUX_DENSE(, false)
