// Team kernels of 2-dimensional even lattices (gc_team_kern.h).
#include "gc_team_inst.h"

#define GC_TEAM_D2(X) X(1, 2, 2) X(2, 2, 2) X(3, 2, 2)
GC_TEAM_DEFINE(d2, GC_TEAM_D2)

// ... and of rings of even length
#define GC_TEAM_D1(X) X(1, 1, 2) X(2, 1, 2) X(3, 1, 2)
GC_TEAM_DEFINE(d1, GC_TEAM_D1)
