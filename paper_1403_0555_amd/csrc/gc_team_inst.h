// Instantiation of the team kernels: GC_TEAM_DEFINE(NAME, LIST) defines the
// entry points of one dimension and number of colours, LIST(X) its classes as
// X(class, d, K).
#pragma once

#include "gc_team_kern.h"

namespace {

template <int D, int K, int CLS, typename R> hipError_t team_occ_t(size_t lds, int block, int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, team_kernel<D, K, CLS, R, 0>, block, lds);
}

template <int D, int K, int CLS, typename R>
hipError_t team_launch_t(int rm, const GcJobDev *jobs, int n_jobs, unsigned long long *job_next, int mmax, int grid,
                         int block, size_t lds, hipStream_t st)
{
#define GC_TEAM_RM(RM)                                                                                             \
    case RM:                                                                                                       \
        hipLaunchKernelGGL((team_kernel<D, K, CLS, R, RM>), dim3(grid), dim3(block), lds, st, jobs, n_jobs,        \
                           job_next, mmax);                                                                        \
        break;
    switch (rm) {
        GC_TEAM_RM(0)
        GC_TEAM_RM(1)
        GC_TEAM_RM(2)
        GC_TEAM_RM(3)
    default: return hipErrorInvalidValue;
    }
#undef GC_TEAM_RM
    return hipGetLastError();
}

}  // namespace

#define GC_TEAM_OCC(CLS, D, K)                                                                                     \
    if (cls == CLS)                                                                                                \
        return f32 ? team_occ_t<D, K, CLS, float>(lds, block, per_cu)                                              \
                   : team_occ_t<D, K, CLS, double>(lds, block, per_cu);
#define GC_TEAM_GO(CLS, D, K)                                                                                      \
    if (cls == CLS)                                                                                                \
        return f32 ? team_launch_t<D, K, CLS, float>(rm, jobs, n_jobs, job_next, mmax, grid, block, lds, st)       \
                   : team_launch_t<D, K, CLS, double>(rm, jobs, n_jobs, job_next, mmax, grid, block, lds, st);
#define GC_TEAM_DEFINE(NAME, LIST)                                                                                 \
    hipError_t gc_team_occupancy_##NAME(int cls, bool f32, size_t lds, int block, int *per_cu)                     \
    {                                                                                                              \
        LIST(GC_TEAM_OCC)                                                                                          \
        return hipErrorInvalidValue;                                                                               \
    }                                                                                                              \
    hipError_t gc_launch_team_##NAME(int cls, bool f32, int rm, const GcJobDev *jobs, int n_jobs,                  \
                                     unsigned long long *job_next, int mmax, int grid, int block, size_t lds,      \
                                     hipStream_t st)                                                               \
    {                                                                                                              \
        LIST(GC_TEAM_GO)                                                                                           \
        return hipErrorInvalidValue;                                                                               \
    }
