// The step's implicit solve.
#define INST_HERE_IMPLICIT
#include "instances.h"

INST_IMPLICIT(, KS)
INST_IMPLICIT(, Flat)
