// Adjoint of the faces and of the implicit solve.
#define INST_HERE_ADJ_FLUX
#define INST_HERE_ADJ_IMPLICIT
#include "instances.h"

INST_ADJ_FLUX(, Dense)
INST_ADJ_IMPLICIT(, Dense)
