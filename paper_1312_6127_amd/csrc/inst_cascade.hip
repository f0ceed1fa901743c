// The grid's full method cascade.
#define INST_HERE_CASCADE
#include "instances.h"

INST_CASCADE(, Dense)
