// The implicit solve of the adjoint's forward step.
#define INST_HERE_IMPLICIT
#include "instances.h"

INST_IMPLICIT(, Dense)
