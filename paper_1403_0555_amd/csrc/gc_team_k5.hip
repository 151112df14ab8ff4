// Team kernels of lattices with five and seven colours (gc_team_kern.h).
#include "gc_team_inst.h"

#define GC_TEAM_K5D2(X) X(2, 2, 5)
#define GC_TEAM_K5D3(X) X(2, 3, 5)
#define GC_TEAM_K5D4(X) X(2, 4, 5)
#define GC_TEAM_K7D2(X) X(2, 2, 7)
#define GC_TEAM_K7D3(X) X(2, 3, 7)
GC_TEAM_DEFINE(k5d2, GC_TEAM_K5D2)
GC_TEAM_DEFINE(k5d3, GC_TEAM_K5D3)
GC_TEAM_DEFINE(k5d4, GC_TEAM_K5D4)
GC_TEAM_DEFINE(k7d2, GC_TEAM_K7D2)
GC_TEAM_DEFINE(k7d3, GC_TEAM_K7D3)
