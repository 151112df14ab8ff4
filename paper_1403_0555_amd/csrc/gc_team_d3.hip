// Team kernels of 3-dimensional even lattices (gc_team_kern.h).
#include "gc_team_inst.h"

#define GC_TEAM_D3(X) X(1, 3, 2) X(2, 3, 2) X(3, 3, 2)
GC_TEAM_DEFINE(d3, GC_TEAM_D3)
