// Wavefront-per-start solver for lattices with even extents (two colours).
//
// Each 64-lane wavefront relaxes one random start with its state resident in
// LDS (at most 64 sites a colour) and never synchronises with other
// wavefronts: a start finishes on its
// own schedule and the wavefront pulls the next start of its job from a
// per-job counter.  The workgroup only synchronises when it moves to another
// job (the orbit's coefficient table may be staged in LDS and is shared by
// its wavefronts).
//
// Layout (colour split, Sec. III checkerboard): site i has colour
// c = (sum_mu x_mu) mod 2 and half index h = i >> 1 (x_0 runs over an even
// extent, so sites 2h and 2h+1 have opposite colours).  A start's state is
// st[c][h] (complex), the update of (c, h) reads its 2d neighbours in
// st[1-c][.], and the orbit supplies per (c, h):
//   nb[c][h]      the 2d neighbour half indices (forward mu = 0..d-1, then backward)
//   coef[c][k][h] U_{i,k} for forward k, conj(U_{i-k,k}) for backward k,
// so that S_i = sum_k coef_k g_{n_k} (eqs. (4)-(5) in the eq. (3) convention).
//
// The stopping norm of sweep t needs div_i on the post-sweep state.  For the
// colour updated last it is formed right after the update; for colour 0 the
// staple S_i of the post-sweep state is exactly the one sweep t+1 computes
// first, so the norm of sweep t is completed there, before sweep t+1's new
// values are written, and the sweep is discarded if the norm has fallen
// below the threshold.  The arithmetic is that of a separate check pass.
#pragma once

#include "gc_common.h"
#include "gc_wave.h"

namespace {

using namespace gc;

// Neighbour half indices of a slot, forward mu = 0..d-1 then backward:
// from its packed table entry (eight 16-bit half indices) ...
struct NbWords {
    u32x4 w;
    __device__ __forceinline__ uint32_t operator()(int k) const
    {
        const uint32_t word = (k >> 1) == 0 ? w.x : (k >> 1) == 1 ? w.y : (k >> 1) == 2 ? w.z : w.w;
        return (k & 1) ? (word >> 16) : (word & 0xFFFFu);
    }
};

// S = sum_k coef_k g_{n_k}, forward mu = 0..d-1 then backward, as in the
// coefficient table, each complex product accumulated by four FMAs.  The
// coefficients come from cf (registers, CF_REG) or from the table at
// coef[(c 2d + k) half + h].
template <int D, typename R, bool CF_REG, typename CP, typename SP, typename NB>
__device__ __forceinline__ typename cx<R>::T staple(const typename cx<R>::T (&cf)[2 * D], CP coef, SP other,
                                                    const NB &nb, int c, int h, int half)
{
    using C = typename cx<R>::T;
    R ax = 0, ay = 0;
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
        const C u = CF_REG ? cf[k] : coef[(c * 2 * D + k) * half + h];
        const C g = other[nb(k)];
        ax = fma(u.x, g.x, ax);
        ax = fma(-u.y, g.y, ax);
        ay = fma(u.x, g.y, ay);
        ay = fma(u.y, g.x, ay);
    }
    C s;
    s.x = ax;
    s.y = ay;
    return s;
}

// The largest volume of a launch's jobs: the stride of the promotion scratch,
// whose regions then stay apart while wavefronts work on different jobs.
__device__ __forceinline__ int max_volume(const GcJobDev *jobs, int n_jobs)
{
    int v = 0;
    for (int j = 0; j < n_jobs; ++j) v = max(v, jobs[j].orb.V);
    return uniform(v);
}

// Synchronisation and reductions over the WPS wavefronts that share a start
// (WPS = 1: one wavefront; otherwise the whole workgroup).  red holds at
// least WPS doubles of LDS.
template <int WPS> __device__ __forceinline__ void start_sync()
{
    if constexpr (WPS > 1) __syncthreads();
    else wave_sync();
}
template <int WPS> __device__ __forceinline__ double start_sum(double v, double *red)
{
    v = wave_sum(v);
    if constexpr (WPS > 1) {
        __syncthreads();   // every wave has read the previous contents of red
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        double t = red[0];
#pragma unroll
        for (int w = 1; w < WPS; ++w) t += red[w];
        v = t;
    }
    return v;
}
template <int WPS> __device__ __forceinline__ double start_max(double v, double *red)
{
    v = wave_max(v);
    if constexpr (WPS > 1) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        double t = red[0];
#pragma unroll
        for (int w = 1; w < WPS; ++w) t = fmax(t, red[w]);
        v = t;
    }
    return v;
}

// Sweeps of one precision on the wave's state st[2][half], at most two slots
// per lane (NS <= 2).  Returns status.  Lane l owns slots h = l + 64k, k < NS,
// of each colour; slots beyond the half volume are computed on a clamped
// index and discarded, so the passes have no divergent branches.  The packed
// neighbour entries and the lane's own values are held in registers, and
// CREG colours (0, 1 or 2, starting with colour 0) keep the coefficients of
// the lane's slots in registers for the whole phase.  Colour 0 of sweep
// t + 1 first reads the colour-0 staples of the state after sweep t; at a
// check point they complete the norm of sweep t.
template <int D, typename R, int NS, bool RELAX, bool MAXABS, bool FULL, int CREG, int WPS, typename CP>
__device__ int relax_wave_t(const GcJobDev &J, const GcWaveOrbit &WO, CP coef, lds_ptr<const u32x4> nbt,
                            lds_ptr<typename cx<R>::T> st, double eps, uint64_t cap, bool fixed, uint64_t &sweeps,
                            double &D_out, double *red)
{
    static_assert(NS <= 2, "register-held neighbour entries");
    const int half = WO.half;
    using C = typename cx<R>::T;
    // thread index within the start: the lane, or the workgroup thread when
    // WPS wavefronts share the start
    const int lane = WPS > 1 ? (int)threadIdx.x : (int)(threadIdx.x & 63);
    lds_ptr<C> st0 = st;
    lds_ptr<C> st1 = st + half;
    const R omega = (R)J.omega;
    // fixed (batch-synchronous pass): the norm only after the last of cap sweeps
    const uint64_t check = fixed ? cap : J.check_every > 0 ? (uint64_t)J.check_every : 1;
    constexpr bool maxabs = MAXABS;
    int hs[NS];
    bool valid[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const int h = lane + 64 * WPS * k;
        valid[k] = FULL || h < half;
        hs[k] = valid[k] ? h : half - 1;
    }
    u32x4 nr[2][NS];
    C own[2][NS];   // the lane's own sites: LDS is only written
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        nr[0][k] = nbt[hs[k]];
        nr[1][k] = nbt[half + hs[k]];
        own[0][k] = st0[hs[k]];
        own[1][k] = st1[hs[k]];
    }
    constexpr int NCR = CREG > 0 ? CREG : 1;
    C cr[NCR][NS][2 * D];
    if constexpr (CREG > 0) {
#pragma unroll
        for (int c = 0; c < CREG; ++c)
#pragma unroll
            for (int k = 0; k < NS; ++k)
#pragma unroll
                for (int q = 0; q < 2 * D; ++q) cr[c][k][q] = coef[(c * 2 * D + q) * half + hs[k]];
    }

    uint64_t t = 0;
    uint64_t until = check;      // sweeps left to the next check point
    bool ckpt = false;           // the state after sweep t is checked
    double part1 = 0.0;          // this lane's colour-1 part of the norm of sweep t
    int status = GC_ST_NONCONVERGED;
    D_out = INFINITY;
    for (;;) {
        const bool pending = (t > 0) && ckpt;
        const bool last = (t == cap);
        // an opaque offset keeps per-slot index arithmetic inside the sweep
        const int z = opaque_zero();
        C gnew[NS];
        double acc0 = 0.0;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int h = hs[k] + z;
            const C s = staple<D, R, (CREG >= 1)>(cr[0][k], coef, st1, NbWords{nr[0][k]}, 0, h, half);
            const C g0 = own[0][k];
            const double dv = (double)fma(g0.x, s.y, -(g0.y * s.x));
            const double a = maxabs ? fmax(acc0, fabs(dv)) : fma(dv, dv, acc0);
            acc0 = valid[k] ? a : acc0;
            gnew[k] = local_update<RELAX, R, !FULL>(g0, s, omega);
        }
        if (pending) {
            // one wave reduction per checked sweep, over both colours' lane parts
            double Dn;
            if (maxabs) Dn = start_max<WPS>(fmax(acc0, part1), red);
            else Dn = start_sum<WPS>(acc0 + part1, red) / (double)(2 * half);
            D_out = Dn;
            if (!(Dn == Dn)) { status = GC_ST_BADNUM; break; }
            if (Dn < eps) {
                status = GC_ST_CONVERGED;
                if (!fixed) break;
            }
        }
        if (last) break;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            own[0][k] = gnew[k];
            if (valid[k]) st0[hs[k]] = gnew[k];
        }
        start_sync<WPS>();
        // ---- colour 1, with its part of the norm of this sweep
        ++t;
        --until;
        ckpt = (until == 0) || (t == cap);
        if (until == 0) until = check;
        const bool chk = ckpt;
        double a1 = 0.0;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int h = hs[k] + z;
            const C s = staple<D, R, (CREG >= 2)>(cr[NCR - 1][k], coef, st0, NbWords{nr[1][k]}, 1, h, half);
            const C g = local_update<RELAX, R, !FULL>(own[1][k], s, omega);
            own[1][k] = g;
            if (valid[k]) st1[hs[k]] = g;
            const double dv = (double)fma(g.x, s.y, -(g.y * s.x));
            const double a = maxabs ? fmax(a1, fabs(dv)) : fma(dv, dv, a1);
            a1 = valid[k] ? a : a1;
        }
        if (chk) part1 = a1;
        start_sync<WPS>();
    }
    sweeps = t;
    return status;
}

// The sweep loop specialised per start (uniform branches): plain relaxation
// or over-relaxation, the max |div| or the mean-square norm, and, for the
// double-precision mean-square sweep, whether every slot lies on the lattice
// (half = 64 WPS NS: no slot is tested and the local update skips the guard
// on the reciprocal square root's argument; the single-precision sweep
// measured slower in that form and keeps the general one).  The variants
// round alike.
template <int D, typename R, int NS, int CREG, int WPS, typename CP>
__device__ int relax_wave(const GcJobDev &J, const GcWaveOrbit &WO, CP coef, lds_ptr<const u32x4> nbt,
                          lds_ptr<typename cx<R>::T> st, double eps, uint64_t cap, bool fixed, uint64_t &sweeps,
                          double &D_out, double *red)
{
#define GC_RW(RELAX, MAXABS, FULL)                                                                         \
    return relax_wave_t<D, R, NS, RELAX, MAXABS, FULL, CREG, WPS>(J, WO, coef, nbt, st, eps, cap, fixed, sweeps, \
                                                                  D_out, red)
    const bool relax = (R)J.omega == (R)1;
    if (J.stop_norm != 0) {
        if (relax) GC_RW(true, true, false);
        GC_RW(false, true, false);
    }
    if (sizeof(R) == 8 && WO.half == 64 * WPS * NS) {
        if (relax) GC_RW(true, false, true);
        GC_RW(false, false, true);
    }
    if (relax) GC_RW(true, false, false);
    GC_RW(false, false, false);
#undef GC_RW
}

template <int D, int NS, int CREG, int CREG32, int WPS, typename CP64, typename CP32>
__device__ void relax_start_wave(const GcJobDev &J, const GcWaveOrbit &WO, CP64 coef64, CP32 coef32,
                                 lds_ptr<const u32x4> nbt, lds_ptr<dbl2> st64, lds_ptr<flt2> st32,
                                 glb_ptr<flt2> bounce, uint64_t local, double *red, RelaxTally &tally)
{
    constexpr int T = 64 * WPS;   // threads on the start
    const int lane = WPS > 1 ? (int)threadIdx.x : (int)(threadIdx.x & 63);
    const GcOrbitDev &O = J.orb;
    const int V = O.V;
    const uint64_t sid = J.first_start + local;

    // random start, written at its colour-split position loc[i]
    for (int b = lane; 4 * b < V; b += T) {
        uint64_t c[4];
        // the caller's start angles, else Philox (the block is skipped then)
        if (!J.theta_init) start_block(J.start_seed, sid, O.orbit_index, (uint64_t)b, c);
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            const int i = 4 * b + k;
            if (i < V) {
                double sn, cs;
                sincos(J.theta_init ? J.theta_init[local * (uint64_t)V + i] : angle_of(c[k]), &sn, &cs);
                const int p = WO.loc[i];
                if (J.precision == 1) st32[p] = flt2{(float)cs, (float)sn};
                else st64[p] = dbl2{cs, sn};
            }
        }
    }
    start_sync<WPS>();

    uint64_t sw32 = 0, sw64 = 0;
    double Dn = INFINITY;
    int status;
    bool in64 = J.precision != 1;
    const bool fixed = (J.flags & GC_JOB_SYNC2) != 0;
    const uint64_t cap = fixed ? (uint64_t)J.fixed_sweeps[local] : J.max_sweeps;
    if (J.precision == 1) {
        status = relax_wave<D, float, NS, CREG32, WPS>(J, WO, coef32, nbt, st32, J.eps32, J.max_sweeps, false, sw32, Dn,
                                                     red);
        if (status == GC_ST_CONVERGED) {
            // promotion g64 = normalise((double) g32): both states share the
            // start's LDS region, so each thread bounces its entries through
            // the start's scratch (it reads back only what it wrote)
            in64 = true;
            for (int p = lane; p < V; p += T) bounce[p] = st32[p];
            start_sync<WPS>();
            for (int p = lane; p < V; p += T) {
                const flt2 g = bounce[p];
                const double xr = (double)g.x, xi = (double)g.y;
                const double r = rsqrt(xr * xr + xi * xi);
                st64[p] = dbl2{xr * r, xi * r};
            }
            start_sync<WPS>();
            status = relax_wave<D, double, NS, CREG, WPS>(J, WO, coef64, nbt, st64, J.eps64, J.max_sweeps, false,
                                                          sw64, Dn, red);
        }
    } else {
        status = relax_wave<D, double, NS, CREG, WPS>(J, WO, coef64, nbt, st64, J.eps64, cap, fixed, sw64, Dn, red);
    }
    // final state in natural site order
    glb_ptr<dbl2> out = as_global(reinterpret_cast<dbl2 *>(J.states + local * (uint64_t)V));
    for (int i = lane; i < V; i += T) {
        const int p = WO.loc[i];
        out[i] = in64 ? st64[p] : dbl2{(double)st32[p].x, (double)st32[p].y};
    }
    if (lane == 0) record_relax(J, local, status, sw32, sw64, Dn, tally);
    start_sync<WPS>();
}

// WG = WAVES wavefronts, one slot per lane and colour (NS = 1).  LDS: [neighbour table
// 16V | coef64 | coef32 when COEF_LDS] then per wave a 16V-byte state region
// (double2[V], or float2[V] in the single-precision phase).
template <int D, int NS, int WAVES, bool COEF_LDS, int CREG>
__global__ __launch_bounds__(64 * WAVES) void wave_kernel(const GcJobDev *__restrict__ jobs,
                                                          const GcWaveOrbit *__restrict__ worbs, int n_jobs,
                                                          unsigned long long *job_next, float2 *bounce_all)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cur_job;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int vmax = max_volume(jobs, n_jobs);
    int j0 = (int)(blockIdx.x % (unsigned)n_jobs);
    for (int round = 0; round < n_jobs; ++round) {
        if (threadIdx.x == 0) {
            int pick = -1;
            for (int k = 0; k < n_jobs; ++k) {
                const int j = (j0 + k) % n_jobs;
                if (__hip_atomic_load(&job_next[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < jobs[j].n_starts) {
                    pick = j;
                    break;
                }
            }
            cur_job = pick;
        }
        __syncthreads();
        const int jn = uniform(cur_job);
        __syncthreads();
        if (jn < 0) break;
        const GcJobDev &J = jobs[jn];
        const GcWaveOrbit &WO = worbs[jn];
        const int V = J.orb.V;
        const int ncoef = 2 * D * V;      // complex entries per precision
        // neighbour table (16 bytes per slot, 16V in all), then the
        // coefficients when staged, then the wavefronts' states
        lds_ptr<u32x4> nbt = as_lds(reinterpret_cast<u32x4 *>(smem));
        {
            glb_ptr<const u32x4> nbg = as_global(reinterpret_cast<const u32x4 *>(WO.nb));
            for (int t = threadIdx.x; t < V; t += 64 * WAVES) nbt[t] = nbg[t];
        }
        size_t off = 16 * (size_t)V;
        const dbl2 *g64 = reinterpret_cast<const dbl2 *>(WO.coef64);
        const flt2 *g32 = reinterpret_cast<const flt2 *>(WO.coef32);
        lds_ptr<dbl2> c64 = as_lds(reinterpret_cast<dbl2 *>(smem + off));
        lds_ptr<flt2> c32 = as_lds(reinterpret_cast<flt2 *>(smem + off + 16 * (size_t)ncoef));
        if (COEF_LDS) {
            for (int t = threadIdx.x; t < ncoef; t += 64 * WAVES) c64[t] = g64[t];
            off += 16 * (size_t)ncoef;
            if (J.precision == 1) {
                for (int t = threadIdx.x; t < ncoef; t += 64 * WAVES) c32[t] = g32[t];
                off += 8 * (size_t)ncoef;
            }
        }
        __syncthreads();
        lds_ptr<dbl2> st64 = as_lds(reinterpret_cast<dbl2 *>(smem + off + (size_t)wave * 16 * V));
        lds_ptr<flt2> st32 = as_lds(reinterpret_cast<flt2 *>(smem + off + (size_t)wave * 16 * V));
        glb_ptr<flt2> bounce =
            as_global(reinterpret_cast<flt2 *>(bounce_all) + ((uint64_t)blockIdx.x * WAVES + wave) * (uint64_t)vmax);
        // Starts are claimed a few at a time, fewer towards the end of the
        // job: a claim is an atomic that all wavefronts wait for in turn.
        const uint64_t n_starts = J.n_starts, waves = (uint64_t)gridDim.x * WAVES;
        RelaxTally tally = {0, 0, 0};
        uint64_t s = 0, end = 0;
        for (;;) {
            if (s == end) {
                const uint64_t left = n_starts - min(end, n_starts);
                const uint64_t chunk = max((uint64_t)1, min((uint64_t)8, left / (4 * waves)));
                unsigned long long c = 0;
                if (lane == 0) c = atomicAdd(&job_next[jn], (unsigned long long)chunk);
                s = uniform((uint64_t)c);
                if (s >= n_starts) break;
                end = min(s + chunk, n_starts);
            }
            lds_ptr<const u32x4> nbc = nbt;
            if (COEF_LDS)
                relax_start_wave<D, NS, CREG, CREG, 1>(J, WO, c64, c32, nbc, st64, st32, bounce, s, nullptr, tally);
            else
                relax_start_wave<D, NS, CREG, CREG, 1>(J, WO, as_global(g64), as_global(g32), nbc, st64, st32, bounce, s,
                                                 nullptr, tally);
            ++s;
        }
        if (lane == 0) flush_tally(J, tally);
        __syncthreads();
        j0 = jn;
    }
}

// One start per workgroup of WPS wavefronts, for lattices above the team
// kernels' (V > 2048): each thread keeps at most two slots per colour, the
// colour passes synchronise the workgroup.  LDS: the neighbour table (16V)
// and one state region (16V).  The coefficients come from the L2, half a
// megabyte per sweep of 8^4 and the bound of it (5.9 us); in single precision
// with 16 wavefronts, where 128 registers allow it, those of colour 0 (up to
// three dimensions all) stay in registers: 10^4 mixed-precision starts of 8^4
// 48.2 -> 44.3 ms, 5000 of 16^3 19.3 -> 17.0, 2000 of 64^2 21.4 -> 19.6.  With
// fewer wavefronts the registers cost workgroups per CU (4^2 x 8^2 in this
// layout took 1.6 to 1.9 times as long).
template <int D, int WPS>
__global__ __launch_bounds__(64 * WPS) void wps_kernel(const GcJobDev *__restrict__ jobs,
                                                       const GcWaveOrbit *__restrict__ worbs, int n_jobs,
                                                       unsigned long long *job_next, float2 *bounce_all)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cur_job;
    __shared__ unsigned long long claim;
    __shared__ double red[WPS];
    __shared__ RelaxTally tally;   // not in registers: the sweeps have none to spare
    const int vmax = max_volume(jobs, n_jobs);
    int j0 = (int)(blockIdx.x % (unsigned)n_jobs);
    for (int round = 0; round < n_jobs; ++round) {
        if (threadIdx.x == 0) {
            int pick = -1;
            for (int k = 0; k < n_jobs; ++k) {
                const int j = (j0 + k) % n_jobs;
                if (__hip_atomic_load(&job_next[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < jobs[j].n_starts) {
                    pick = j;
                    break;
                }
            }
            cur_job = pick;
        }
        __syncthreads();
        const int jn = uniform(cur_job);
        __syncthreads();
        if (jn < 0) break;
        const GcJobDev &J = jobs[jn];
        const GcWaveOrbit &WO = worbs[jn];
        const int V = J.orb.V;
        lds_ptr<u32x4> nbt = as_lds(reinterpret_cast<u32x4 *>(smem));
        glb_ptr<const u32x4> nbg = as_global(reinterpret_cast<const u32x4 *>(WO.nb));
        for (int t = threadIdx.x; t < V; t += 64 * WPS) nbt[t] = nbg[t];
        __syncthreads();
        lds_ptr<dbl2> st64 = as_lds(reinterpret_cast<dbl2 *>(smem + 16 * (size_t)V));
        lds_ptr<flt2> st32 = as_lds(reinterpret_cast<flt2 *>(smem + 16 * (size_t)V));
        glb_ptr<flt2> bounce = as_global(reinterpret_cast<flt2 *>(bounce_all) + (uint64_t)blockIdx.x * (uint64_t)vmax);
        const dbl2 *g64 = reinterpret_cast<const dbl2 *>(WO.coef64);
        const flt2 *g32 = reinterpret_cast<const flt2 *>(WO.coef32);
        lds_ptr<const u32x4> nbc = nbt;
        if (threadIdx.x == 0) tally = RelaxTally{0, 0, 0};
        for (;;) {
            if (threadIdx.x == 0) claim = atomicAdd(&job_next[jn], 1ULL);
            __syncthreads();
            const uint64_t s = uniform((uint64_t)claim);
            __syncthreads();
            if (s >= J.n_starts) break;
            relax_start_wave<D, 2, 0, WPS < 16 ? 0 : D <= 3 ? 2 : 1, WPS>(J, WO, as_global(g64), as_global(g32), nbc, st64, st32, bounce, s, red,
                                        tally);
        }
        if (threadIdx.x == 0) flush_tally(J, tally);
        __syncthreads();
        j0 = jn;
    }
}

template <int D, int WPS>
hipError_t wps_launch_t(const GcJobDev *jobs, const GcWaveOrbit *worbs, int n_jobs, unsigned long long *job_next,
                        float2 *bounce, int grid, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL((wps_kernel<D, WPS>), dim3(grid), dim3(64 * WPS), lds, s, jobs, worbs, n_jobs, job_next,
                       bounce);
    return hipGetLastError();
}

template <int D, int WPS>
hipError_t wps_occ_t(size_t lds, int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, wps_kernel<D, WPS>, 64 * WPS, lds);
}

template <int D, int NS, int WAVES, bool CL, int CREG>
hipError_t launch_v(const GcJobDev *jobs, const GcWaveOrbit *worbs, int n_jobs, unsigned long long *job_next,
                    float2 *bounce, int grid, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL((wave_kernel<D, NS, WAVES, CL, CREG>), dim3(grid), dim3(64 * WAVES), lds, s, jobs, worbs,
                       n_jobs, job_next, bounce);
    return hipGetLastError();
}

template <int D, int NS, int WAVES, bool CL, int CREG>
hipError_t occ_v(size_t lds, int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, wave_kernel<D, NS, WAVES, CL, CREG>, 64 * WAVES, lds);
}

// Register-held coefficients: creg 1 holds colour 0, creg 2 both colours.
template <int D, int NS, int WAVES>
hipError_t launch_t(const GcJobDev *jobs, const GcWaveOrbit *worbs, int n_jobs, unsigned long long *job_next,
                    int variant, float2 *bounce, int grid, size_t lds, hipStream_t s)
{
    const bool cl = (variant & 1) != 0;
    switch (variant >> 1) {
    case 0:
        return cl ? launch_v<D, NS, WAVES, true, 0>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s)
                  : launch_v<D, NS, WAVES, false, 0>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);
    case 1:
        return cl ? launch_v<D, NS, WAVES, true, 1>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s)
                  : launch_v<D, NS, WAVES, false, 1>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);
    case 2:
        return cl ? launch_v<D, NS, WAVES, true, 2>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s)
                  : launch_v<D, NS, WAVES, false, 2>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);
    default: return hipErrorInvalidValue;
    }
}

template <int D, int NS, int WAVES>
hipError_t occ_t(int variant, size_t lds, int *per_cu)
{
    const bool cl = (variant & 1) != 0;
    switch (variant >> 1) {
    case 0: return cl ? occ_v<D, NS, WAVES, true, 0>(lds, per_cu) : occ_v<D, NS, WAVES, false, 0>(lds, per_cu);
    case 1: return cl ? occ_v<D, NS, WAVES, true, 1>(lds, per_cu) : occ_v<D, NS, WAVES, false, 1>(lds, per_cu);
    case 2: return cl ? occ_v<D, NS, WAVES, true, 2>(lds, per_cu) : occ_v<D, NS, WAVES, false, 2>(lds, per_cu);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Entry points of one lattice dimension D: each gc_waveD.hip instantiates
// the kernels of its D only.
#define GC_WAVE_DEFINE_DIM(D)                                                                             \
    hipError_t gc_wave_occupancy_d##D(int variant, size_t lds, int *per_cu)                                \
    {                                                                                                     \
        return occ_t<D, 1, GC_WAVES>(variant, lds, per_cu);                                               \
    }                                                                                                     \
    hipError_t gc_launch_wave_d##D(const GcJobDev *jobs, const GcWaveOrbit *worbs, int n_jobs,            \
                                   unsigned long long *job_next, int variant, float2 *bounce, int grid,   \
                                   size_t lds, hipStream_t s)                                             \
    {                                                                                                     \
        return launch_t<D, 1, GC_WAVES>(jobs, worbs, n_jobs, job_next, variant, bounce, grid, lds, s);    \
    }                                                                                                     \
    hipError_t gc_wps_occupancy_d##D(int wps, size_t lds, int *per_cu)                                    \
    {                                                                                                     \
        switch (wps) {                                                                                    \
        case 2: return wps_occ_t<D, 2>(lds, per_cu);                                                      \
        case 4: return wps_occ_t<D, 4>(lds, per_cu);                                                      \
        case 6: return wps_occ_t<D, 6>(lds, per_cu);                                                      \
        case 8: return wps_occ_t<D, 8>(lds, per_cu);                                                      \
        case 16: return wps_occ_t<D, 16>(lds, per_cu);                                                    \
        default: return hipErrorInvalidValue;                                                             \
        }                                                                                                 \
    }                                                                                                     \
    hipError_t gc_launch_wps_d##D(int wps, const GcJobDev *jobs, const GcWaveOrbit *worbs, int n_jobs,   \
                                  unsigned long long *job_next, float2 *bounce, int grid, size_t lds,     \
                                  hipStream_t s)                                                          \
    {                                                                                                     \
        switch (wps) {                                                                                    \
        case 2: return wps_launch_t<D, 2>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);          \
        case 4: return wps_launch_t<D, 4>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);          \
        case 6: return wps_launch_t<D, 6>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);          \
        case 8: return wps_launch_t<D, 8>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);          \
        case 16: return wps_launch_t<D, 16>(jobs, worbs, n_jobs, job_next, bounce, grid, lds, s);        \
        default: return hipErrorInvalidValue;                                                             \
        }                                                                                                 \
    }
