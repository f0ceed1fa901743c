// The batched implicit solve.
#define INST_HERE_BATCH
#include "instances.h"

INST_BATCH(, Dense)
