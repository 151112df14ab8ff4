// Wavefront-per-start and workgroup-per-start relax kernels of 2-dimensional
// lattices (see gc_wave_kern.h); one translation unit per dimension.
#include "gc_wave_kern.h"

GC_WAVE_DEFINE_DIM(2)
