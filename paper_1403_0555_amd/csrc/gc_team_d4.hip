// Team kernels of 4-dimensional even lattices (gc_team_kern.h).
#include "gc_team_inst.h"

#define GC_TEAM_D4(X) X(1, 4, 2) X(2, 4, 2) X(3, 4, 2) X(4, 4, 2) X(5, 4, 2)
GC_TEAM_DEFINE(d4, GC_TEAM_D4)
