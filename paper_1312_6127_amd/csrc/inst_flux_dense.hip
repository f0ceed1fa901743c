// Face fluxes in the dense form: FP32, and FP64 for the Courant step and the adjoint.
#define INST_HERE_FLUX
#define INST_HERE_FLUX_F32
#include "instances.h"

INST_FLUX(, Dense)
INST_FLUX_F32(, Dense)
