// Team kernels of lattices with three colours (gc_team_kern.h).
#include "gc_team_inst.h"

#define GC_TEAM_K3D2(X) X(1, 2, 3) X(2, 2, 3)
#define GC_TEAM_K3D3(X) X(1, 3, 3) X(2, 3, 3)
#define GC_TEAM_K3D4(X) X(2, 4, 3)
GC_TEAM_DEFINE(k3d2, GC_TEAM_K3D2)
GC_TEAM_DEFINE(k3d3, GC_TEAM_K3D3)
GC_TEAM_DEFINE(k3d4, GC_TEAM_K3D4)
