// Team relaxation kernels (gc_team_kern.h): shapes and launch entry points.
#pragma once

#include "gc_internal.h"

// An instantiation: spt sites of each colour per thread, m starts in step, at
// most maxw wavefronts per workgroup, compiled for minw wavefronts per SIMD
// (512 / minw registers), pf neighbours fetched ahead; lone: a start left on
// its own has a loop of its own, in double precision.
struct GcTeamClass {
    int spt, m, maxw, minw, pf;
    bool lone;
};

// Classes by dimension and colours.  The links and neighbour offsets of a
// thread's sites, 10 d K registers, set the register budget, the budget the
// wavefronts per SIMD, and the LDS of 160 KiB the starts in step.  Measured,
// 10^9 site updates per second at 100 sweeps of 10^5 starts (over-relaxed,
// double precision, the start states drawn within the time), against the
// kernels these replaced (a wavefront, or with odd extents a workgroup, per
// start): 6^4 284 against 270, 4^2 x 8^2 312 against 234, 10^3 403 against
// 333, 8^3 403 against 315, 12^3 354 against 215, 32^2 487 against 306, 4^4
// 307 against 175, 16^2 439 against 405, 9^3 284 against 80; and a sweep of a
// single start: 6^4 1.5 against 6.0 us, 4^2 x 8^2 0.9 against 6.0, 10^3 1.2
// against 3.7, 12^3 1.6 against 10.6, 9^3 1.4 against 6.1.  7^2 is the one
// lattice found slower in bulk (1.5 10^5 starts 20.4 against 18.4 ms; fewer
// starts and plain relaxation are faster): 140 registers of links leave two
// wavefronts a SIMD, and held to three they spill.  The clock falls from 2.2 to
// 1.9 GHz as the vector units fill: the power limit takes part of what a
// better overlap would give.
// The lone starts' loop costs the main one some registers: none where there
// are enough, but with it 200 sweeps of 5 10^4 starts of 10^3 took 30.0 ms
// (23.8), of 2 10^4 of 12^3 22.2 (18.8) and of 3 10^4 of 6^4 27.9 (26.5), so
// those classes do without (single precision has room in all).
// Four dimensions, eight wavefronts: seven starts in step do not fit, and five
// take less than three with the registers of the next class (4^2 x 8^2, 200
// starts 0.74 against 0.90 ms, 5000 4.7 against 5.2, 60000 39.1 against 39.5).
constexpr GcTeamClass gc_team_class(int d, int K, int cls)
{
    if (K == 2) {
        if (d <= 2)
            return cls == 1   ? GcTeamClass{1, 3, 4, 4, 2 * d, true}
                   : cls == 2 ? GcTeamClass{1, 3, 8, 4, 2 * d, true}
                              : GcTeamClass{1, 3, 16, 4, 2 * d, true};
        if (d == 3)
            return cls == 1   ? GcTeamClass{1, 3, 4, 3, 4, true}
                   : cls == 2 ? GcTeamClass{1, 3, 8, 4, 1, false}
                              : GcTeamClass{1, 3, 16, 4, 1, false};
        return cls == 1   ? GcTeamClass{1, 3, 4, 3, 0, true}
               : cls == 2 ? GcTeamClass{1, 7, 8, 2, 4, true}
               : cls == 3 ? GcTeamClass{1, 5, 8, 2, 4, true}
               : cls == 4 ? GcTeamClass{1, 3, 12, 3, 1, false}
                          : GcTeamClass{2, 3, 8, 2, 1, false};
    }
    if (K == 3 && d == 2) return cls == 1 ? GcTeamClass{1, 3, 4, 4, 0, true} : GcTeamClass{1, 3, 8, 4, 0, true};
    if (K == 3 && d == 3) return cls == 1 ? GcTeamClass{1, 3, 4, 3, 0, true} : GcTeamClass{1, 3, 8, 2, 0, true};
    return GcTeamClass{1, 3, 8, 2, 0, true};
}

// Shape of the team kernel for a lattice: its class (0: none, the other relax
// kernels take the lattice) and the wavefronts per workgroup.
struct GcTeamShape {
    int cls, waves;
};
GcTeamShape gc_team_shape(int d, int K, int V);

// LDS: m states with a place per thread and colour, the norm's partial sums
// (of the last colour apart with two colours), the positions of the V sites.
constexpr size_t gc_team_lds_bytes(int d, int K, const GcTeamShape &s, int V, bool f32)
{
    const GcTeamClass c = gc_team_class(d, K, s.cls);
    return (size_t)64 * s.waves * c.m * ((f32 ? 8 : 16) * K * c.spt + (K == 2 ? 16 : 8)) + 2 * (size_t)V;
}

// f32: the single-precision phase of a mixed launch (converged starts are
// promoted into their state row for the double-precision launch that
// follows); rm: bit 0 plain relaxation, bit 1 the max |div| norm; mmax: the
// most starts a workgroup takes at once (1 .. m).
hipError_t gc_team_occupancy(int d, int K, const GcTeamShape &s, bool f32, size_t lds, int *per_cu);
hipError_t gc_launch_team(int d, int K, const GcTeamShape &s, bool f32, int rm, const GcJobDev *jobs, int n_jobs,
                          unsigned long long *job_next, int mmax, int grid, size_t lds, hipStream_t st);
