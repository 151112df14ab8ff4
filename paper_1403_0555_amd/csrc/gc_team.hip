// Shapes and dispatch of the team relaxation kernels (gc_team_kern.h); the
// kernels are instantiated in gc_team_d2.hip .. gc_team_k5.hip.
#include "gc_team.h"

GcTeamShape gc_team_shape(int d, int K, int V)
{
    const GcTeamShape none = {0, 0};
    const int w = (V / K + 63) / 64;   // wavefronts at one site of a colour per thread
    if (K == 2) {
        // up to 64 sites per colour one wavefront holds the whole start:
        // wave_kernel (gc_wave_kern.h) needs no barrier and takes 0.6 us for a
        // single start's sweep of 8^2 against 0.95, at the same rate in bulk
        if (w <= 1) return none;
        if (w <= 4) return {1, w};
        if (d < 4) return w <= 8 ? GcTeamShape{2, w} : w <= 16 ? GcTeamShape{3, w} : none;
        // four dimensions: 80 registers of links and offsets a site and
        // colour leave room for 12 wavefronts of one site or 8 of two; seven
        // starts of seven wavefronts are 149 KB of LDS, of eight 170
        if (w <= 7) return {2, w};
        return w == 8 ? GcTeamShape{3, w} : w <= 12 ? GcTeamShape{4, w} : w <= 16 ? GcTeamShape{5, (w + 1) / 2} : none;
    }
    if (d < 2) return none;
    if (K == 3) return w <= 4 && d < 4 ? GcTeamShape{1, w} : w <= 8 ? GcTeamShape{2, w} : none;
    if (K == 5) return w <= 8 ? GcTeamShape{2, w} : none;
    // seven colours: 280 registers in four dimensions; three starts of seven
    // wavefronts are 163 KB of LDS
    if (K == 7 && d < 4) return w <= 6 ? GcTeamShape{2, w} : none;
    return none;
}

#define GC_TEAM_DECLARE(NAME)                                                                                    \
    hipError_t gc_team_occupancy_##NAME(int cls, bool f32, size_t lds, int block, int *per_cu);                  \
    hipError_t gc_launch_team_##NAME(int cls, bool f32, int rm, const GcJobDev *jobs, int n_jobs,                \
                                     unsigned long long *job_next, int mmax, int grid, int block, size_t lds,    \
                                     hipStream_t st);
GC_TEAM_DECLARE(d1)
GC_TEAM_DECLARE(d2)
GC_TEAM_DECLARE(d3)
GC_TEAM_DECLARE(d4)
GC_TEAM_DECLARE(k3d2)
GC_TEAM_DECLARE(k3d3)
GC_TEAM_DECLARE(k3d4)
GC_TEAM_DECLARE(k5d2)
GC_TEAM_DECLARE(k5d3)
GC_TEAM_DECLARE(k5d4)
GC_TEAM_DECLARE(k7d2)
GC_TEAM_DECLARE(k7d3)

#define GC_TEAM_SWITCH(FN, ...)                                                                                  \
    switch (10 * K + d) {                                                                                        \
    case 21: return FN##_d1(__VA_ARGS__);                                                                        \
    case 22: return FN##_d2(__VA_ARGS__);                                                                        \
    case 23: return FN##_d3(__VA_ARGS__);                                                                        \
    case 24: return FN##_d4(__VA_ARGS__);                                                                        \
    case 32: return FN##_k3d2(__VA_ARGS__);                                                                      \
    case 33: return FN##_k3d3(__VA_ARGS__);                                                                      \
    case 34: return FN##_k3d4(__VA_ARGS__);                                                                      \
    case 52: return FN##_k5d2(__VA_ARGS__);                                                                      \
    case 53: return FN##_k5d3(__VA_ARGS__);                                                                      \
    case 54: return FN##_k5d4(__VA_ARGS__);                                                                      \
    case 72: return FN##_k7d2(__VA_ARGS__);                                                                      \
    case 73: return FN##_k7d3(__VA_ARGS__);                                                                      \
    default: return hipErrorInvalidValue;                                                                        \
    }

hipError_t gc_team_occupancy(int d, int K, const GcTeamShape &s, bool f32, size_t lds, int *per_cu)
{
    GC_TEAM_SWITCH(gc_team_occupancy, s.cls, f32, lds, 64 * s.waves, per_cu)
}

hipError_t gc_launch_team(int d, int K, const GcTeamShape &s, bool f32, int rm, const GcJobDev *jobs, int n_jobs,
                          unsigned long long *job_next, int mmax, int grid, size_t lds, hipStream_t st)
{
    GC_TEAM_SWITCH(gc_launch_team, s.cls, f32, rm, jobs, n_jobs, job_next, mmax, grid, 64 * s.waves, lds, st)
}
