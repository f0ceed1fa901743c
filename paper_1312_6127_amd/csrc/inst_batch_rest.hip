// The batched solve's full method cascade.
#define INST_HERE_BATCH_REST
#include "instances.h"

INST_BATCH_REST(, Dense)
