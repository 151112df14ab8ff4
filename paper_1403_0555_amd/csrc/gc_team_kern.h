// Relaxation by a team of wavefronts: one workgroup holds its orbit's links
// in registers and relaxes up to M random starts in step, their states side
// by side in LDS.
//
// Thread j owns site j (and j + blockDim.x, SPT = 2) of every colour.  Its
// 2d link coefficients and neighbour positions per colour are loaded once per
// orbit and serve every sweep of every start: a site update reads its 2d
// neighbours and its own value from LDS and nothing else, against a
// neighbour entry, 2d links and the exchange of colours besides where a
// wavefront holds a start on its own.  What bounds it is the vector unit: 63
// to 70 vector instructions per site update in four dimensions (32 of them
// the staple's FMAs) and 9 16-byte LDS reads (217 bytes per cycle and CU
// measured: 42 cycles per 64 sites against the 70 of the vector units); on
// 6^4 the SIMDs issue vector instructions in about 60 % of the cycles, the
// rest goes to the two barriers of a sweep.  The M starts share the barriers,
// and a workgroup left with one start spends all its wavefronts on it, so a
// launch of few starts, or the slowest starts of a long one, run at a latency
// of a few thousand cycles per sweep (6^4: 1.5 us against 6.0 us for a
// wavefront on its own).  With the drawing of their start states, 10^6 starts
// of 6^4 relax in 562 ms (599 ms in the wavefront-per-start layout on the same
// machine), 10^5 of 10^3 in 27.9 ms (36.1), 10^4 of 9^3 in 5.2 ms (19.1).
//
// LDS: X[p][m], the M starts' values of the site at colour-sorted position p
// (colour c's sites at c V/K + rank, ascending), then red[m][thread] (the
// stopping norm's partial sums), then inv[i], the position of site i.  M is
// odd: the 16 M byte stride between neighbouring sites then spreads a
// wavefront's accesses over the banks.
//
// Sweep t's norm takes, for the colour updated last, the staple that update
// used (its neighbours have their final values by then), for colour 0 the
// staple that sweep t + 1 starts with, and a staple pass of its own for the
// colours between (K > 2).
#pragma once

#include "gc_common.h"
#include "gc_team.h"

#include <type_traits>

namespace {

using namespace gc;

// f(0), ..., f(N - 1) with the index a compile-time constant: what it indexes
// stays in registers.
template <int N, int I = 0, typename F> __device__ __forceinline__ void each(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each<N, I + 1>(f);
    }
}

// S += u g.  Two colours: four chained FMAs per product; odd colourings:
// each product rounded on its own, then added (the order of the generic
// kernel in gc_relax_wg.hip).
template <int K, typename R, typename C> __device__ __forceinline__ void team_mad(R &ax, R &ay, const C &u, const C &g)
{
    if constexpr (K == 2) {
        ax = fma(u.x, g.x, ax);
        ax = fma(-u.y, g.y, ax);
        ay = fma(u.x, g.y, ay);
        ay = fma(u.y, g.x, ay);
    } else {
#pragma clang fp contract(off)
        ax = ax + fma(u.x, g.x, -(u.y * g.y));
        ay = ay + fma(u.x, g.y, u.y * g.x);
    }
}

// local_update (gc_common.h) with the case |S| = 0, which leaves g unchanged,
// in a branch of its own that hardly any wavefront takes: four selects fewer
// per site.
template <bool RELAX, typename R>
__device__ __forceinline__ typename cx<R>::T team_update(typename cx<R>::T g0, typename cx<R>::T s, R omega)
{
    typename cx<R>::T g = local_update<RELAX, R, false, false>(g0, s, omega);
    const bool zero = !(fma(s.y, s.y, s.x * s.x) > (R)0);
    if (__builtin_expect(__any(zero), 0)) {
        g.x = zero ? g0.x : g.x;
        g.y = zero ? g0.y : g.y;
    }
    return g;
}

// What the workgroup knows of its M starts.
template <int M> struct TeamShared {
    unsigned long long local[M];   // index in the job
    double sum[M];                 // the norm's sum over the sites
    double lone[6];                // norms of a lone start's sweeps
    double D[M];                   // of a start that stops: its norm,
    int32_t status[M];             // status
    uint32_t sweeps[M];            // and sweeps
    uint32_t born[M], end[M];      // the team's sweep count at its begin and at its cap
    uint32_t near;                 // starts that may have stopped (none in most sweeps)
    int32_t spare;                 // a start is claimed ahead
    RelaxTally tally;
};

template <int D, int K, int SPT, int M, int MAXW, int PF, bool LONE, typename R, bool RELAX, bool MAXABS>
__device__ __forceinline__ void team_job(const GcJobDev &J, unsigned long long *next, int mmax, unsigned char *smem,
                                         TeamShared<M> &sh)
{
    using C = typename cx<R>::T;
    constexpr bool F32 = sizeof(R) == 4;
    constexpr uint32_t SZ = (uint32_t)sizeof(C);
    const int V = uniform(J.orb.V), nc = V / K;
    const int tid = (int)threadIdx.x, B = (int)blockDim.x;
    const int lane = tid & 63, wave = uniform(tid >> 6), waves = B >> 6;
    const int sites = K * B * SPT;   // a place for every thread and colour
    lds_ptr<C> X = as_lds(reinterpret_cast<C *>(smem));
    lds_ptr<double> red = as_lds(reinterpret_cast<double *>(smem + (size_t)SZ * M * sites));   // [m][thread]
    lds_ptr<double> red1 = red + M * B;   // two colours: the part from the colour updated last
    lds_ptr<uint16_t> inv = (lds_ptr<uint16_t>)(red + (K == 2 ? 2 : 1) * M * B);
    lds_ptr<unsigned char> xb = (lds_ptr<unsigned char>)X;
    const R omega = (R)J.omega;
    const double eps = F32 ? J.eps32 : J.eps64;
    const bool fixed = !F32 && (uniform((int)J.flags) & GC_JOB_SYNC2) != 0;
    const bool from32 = !F32 && (uniform((int)J.flags) & GC_JOB_FROM32) != 0;
    const uint32_t check = uniform(J.check_every) > 0 ? (uint32_t)uniform(J.check_every) : 1u;
    const bool every = check == 1 && !fixed;
    // a sum of norms at least this is not below eps (a margin for rounding)
    const double far = MAXABS ? eps : eps * (double)V * (1.0 + 1e-14);

    // positions, links and neighbours of the thread's sites; a thread
    // without a site of its own has a place that is its own only neighbour,
    // g = S = 1: it stays so and adds nothing to the norm
    for (int r = tid; r < V; r += B) {
        const int c = r / nc;
        inv[J.orb.perm[r]] = (uint16_t)(r + c * (B * SPT - nc));
    }
    for (int x = tid; x < M * sites; x += B) X[x] = C{1, 0};
    __syncthreads();
    const uint32_t own = SZ * M * (uint32_t)tid;   // of colour 0, s = 0
    uint32_t off[K][SPT][2 * D];
    C cf[K][SPT][2 * D];
    auto load_links = [&]() __attribute__((always_inline)) {
        const int z = opaque_zero();   // loaded anew each time
#pragma unroll
        for (int c = 0; c < K; ++c)
#pragma unroll
            for (int s = 0; s < SPT; ++s) {
                const int j = tid + B * s;
                const int i = J.orb.perm[c * nc + min(j, nc - 1) + z];
#pragma unroll
                for (int k = 0; k < 2 * D; ++k) {
                    // two colours: forward mu = 0..d-1, then backward; odd
                    // colourings: forward and backward by turns
                    const int mu = K == 2 ? (k < D ? k : k - D) : k / 2;
                    const bool fw = K == 2 ? k < D : (k & 1) == 0;
                    const int n = J.orb.nbr[(fw ? mu : D + mu) * V + i];
                    off[c][s][k] = SZ * M * (j < nc ? (uint32_t)inv[n] : (uint32_t)(tid + B * (c * SPT + s)));
                    const C u = F32 ? as_global(reinterpret_cast<const C *>(J.orb.U32))[mu * V + (fw ? i : n)]
                                    : as_global(reinterpret_cast<const C *>(J.orb.U64))[mu * V + (fw ? i : n)];
                    cf[c][s][k].x = j < nc ? u.x : k == 0 ? (R)1 : (R)0;
                    cf[c][s][k].y = j < nc ? (fw ? u.y : -u.y) : (R)0;
                }
            }
    };
    load_links();

    uint32_t T = 0;             // the team's sweeps
    uint32_t act = 0;           // places taken (the masks are the same in every lane)
    uint32_t fresh = 0;         // ... by starts without a sweep yet
    bool exhausted = false;
    const uint32_t all = (1u << mmax) - 1u;
    C old[K == 2 ? 2 : 1][M][SPT];   // two colours: both before the sweep in progress; else colour 0 after it

    auto gather = [&](int c, int s, int m, int k) __attribute__((always_inline)) {
        return *(lds_ptr<const C>)(xb + off[c][s][k] + SZ * m);
    };
    auto site = [&](int c, int s, int m) __attribute__((always_inline)) {
        return (lds_ptr<C>)(xb + (own + SZ * M * (uint32_t)(B * (c * SPT + s))) + SZ * m);
    };
    // the first PF neighbours from pf, the others loaded here
    auto staple = [&](int c, int s, int m, const C *pf) __attribute__((always_inline)) {
        R ax = 0, ay = 0;
#pragma unroll
        for (int k = 0; k < 2 * D; ++k) team_mad<K>(ax, ay, cf[c][s][k], (pf && k < PF) ? pf[k] : gather(c, s, m, k));
        C r;
        r.x = ax;
        r.y = ay;
        return r;
    };
    // f(m, s, prefetched neighbours) for the sites of colour c of the starts
    // in mask: with every place taken, the next site's first PF neighbours
    // are on their way while f works on this one
    auto pass = [&](auto cc, uint32_t mask, auto f) __attribute__((always_inline)) {
        constexpr int c = decltype(cc)::value;
        if (__builtin_expect(mask == (1u << M) - 1u, 1)) {
            C pf[2][PF > 0 ? PF : 1];
#pragma unroll
            for (int k = 0; k < PF; ++k) pf[0][k] = gather(c, 0, 0, k);
            each<M * SPT>([&](auto qc) __attribute__((always_inline)) {
                constexpr int q = decltype(qc)::value, nx = q + 1;
                if constexpr (nx < M * SPT && PF > 0) {
#pragma unroll
                    for (int k = 0; k < PF; ++k) pf[nx & 1][k] = gather(c, nx % SPT, nx / SPT, k);
                    __builtin_amdgcn_sched_barrier(0);
                }
                f(std::integral_constant<int, q / SPT>{}, std::integral_constant<int, q % SPT>{},
                  PF > 0 ? pf[q & 1] : (const C *)nullptr);
            });
        } else {
            each<M * SPT>([&](auto qc) __attribute__((always_inline)) {
                constexpr int q = decltype(qc)::value;
                if ((mask >> (q / SPT)) & 1u)
                    f(std::integral_constant<int, q / SPT>{}, std::integral_constant<int, q % SPT>{}, (const C *)nullptr);
            });
        }
    };
    // |div|^2 (or |div|) of one more site
    auto norm = [&](double acc, const C &g, const C &s) __attribute__((always_inline)) {
        const double dv = (double)fma(g.x, s.y, -(g.y * s.x));
        return MAXABS ? fmax(acc, fabs(dv)) : fma(dv, dv, acc);
    };
    // The wavefronts that add up the norms: first those of the SIMDs that hold
    // one wavefront fewer (w mod 4 >= waves mod 4), which wait at the barriers
    // otherwise, then the rest; mine: the starts of this one.
    uint32_t mine = 0;
    {
        const int r = waves & 3, light = (4 - r) * (waves >> 2);
        for (int m = 0; m < M; ++m) {
            const int k = m % waves, h = k - light;
            const int w = k < light ? 4 * (k / (4 - r)) + r + k % (4 - r) : 4 * (h / r) + h % r;
            if (w == wave) mine |= 1u << m;
        }
    }
    auto reduce = [&](uint32_t mask) __attribute__((always_inline)) {
        for (uint32_t left = mask & mine; left; left &= left - 1) {
            const int m = __builtin_ctz(left);
            double x[MAXW];
#pragma unroll
            for (int q = 0; q < MAXW; ++q) x[q] = red[m * B + 64 * min(q, waves - 1) + lane];
            double v = x[0];
#pragma unroll
            for (int q = 1; q < MAXW; ++q) {
                const double y = q < waves ? x[q] : 0.0;
                v = MAXABS ? fmax(v, y) : v + y;
            }
            v = MAXABS ? wave_max(v) : wave_sum(v);
            // not below eps for sure, and not at the cap: the start goes on
            if (lane == 0) {
                sh.sum[m] = v;
                if (!(v >= far) || T == sh.end[m]) atomicOr(&sh.near, 1u << m);
            }
        }
    };
    // starts whose norm after their last sweep is due
    auto due = [&]() __attribute__((always_inline)) {
        if (every) return act & ~fresh;
        const uint32_t t = T - sh.born[lane < M ? lane : 0];
        const bool is = lane < M && (((act & ~fresh) >> lane) & 1u) &&
                        (T == sh.end[lane < M ? lane : 0] || (!fixed && t % check == 0));
        return (uint32_t)uniform((int)__ballot(is));
    };
    // of the starts in near, those that stop after their last sweep: the norm
    // is below eps, not a number, or taken at the cap.  Lane m looks at
    // start m; every wavefront writes the same.
    auto decide = [&](uint32_t near) __attribute__((always_inline)) {
        const double v = sh.sum[lane < M ? lane : 0];
        const double Dn = MAXABS ? v : v / (double)V;
        const bool bad = !(Dn == Dn), conv = Dn < eps;
        const bool stop =
            lane < M && ((near >> lane) & 1u) && (bad || (conv && !fixed) || T == sh.end[lane < M ? lane : 0]);
        if (stop) {
            sh.D[lane] = Dn;
            sh.status[lane] = bad ? GC_ST_BADNUM : conv ? GC_ST_CONVERGED : GC_ST_NONCONVERGED;
            sh.sweeps[lane] = T - sh.born[lane];
        }
        __syncthreads();
        if (tid == 0) sh.near = 0;
        return (uint32_t)uniform((int)__ballot(stop));
    };
    // final states (X) and records of the starts in fin, which leave their
    // places
    auto finish = [&](uint32_t fin) __attribute__((always_inline)) {
        for (uint32_t left = fin; left; left &= left - 1) {
            const int m = __builtin_ctz(left);
            const uint64_t loc = uniform((uint64_t)sh.local[m]);
            const int status = uniform(sh.status[m]);
            glb_ptr<dbl2> out = as_global(reinterpret_cast<dbl2 *>(J.states + loc * (uint64_t)V));
            const bool promote = F32 && status == GC_ST_CONVERGED;
            for (int i = tid; i < V; i += B) {
                const C g = X[M * inv[i] + m];
                const double xr = (double)g.x, xi = (double)g.y;
                const double r = promote ? rsqrt(xr * xr + xi * xi) : 1.0;
                out[i] = promote ? dbl2{xr * r, xi * r} : dbl2{xr, xi};
            }
            if (tid == 0) {
                const uint32_t sweeps = sh.sweeps[m];
                if (promote) {
                    // its double-precision phase is the next launch's
                    GcStartRec r = {};
                    r.status = GC_ST_PROMOTED;
                    r.sweeps32 = sweeps;
                    r.D = sh.D[m];
                    r.lambda2 = NAN;
                    J.rec[loc] = r;
                } else {
                    const uint32_t sw32 = from32 ? J.rec[loc].sweeps32 : 0u;
                    record_relax(J, loc, status, F32 ? sweeps : sw32, F32 ? 0 : sweeps, sh.D[m], sh.tally);
                }
            }
        }
        act &= ~fin;
    };
    // A new start for every free place, the first of them one claimed ahead
    // while many are left: the answer to its atomic is there by then.
    unsigned long long ahead = ~0ULL;   // wavefront 0, lane 0; ~0: none
    bool spare = false;                 // one is claimed ahead
    auto refill = [&]() __attribute__((always_inline)) {
        const uint64_t n_starts = J.n_starts;
        __syncthreads();   // nobody reads the places or their entries in sh any more
        if (wave == 0) {
            const uint64_t held = uniform((uint64_t)ahead);
            const int first = __builtin_ctz(~act);
            unsigned long long s = 0;
            if (lane < mmax && !((act >> lane) & 1u)) {
                s = (lane == first && spare) ? held : atomicAdd(next, 1ULL);
                // finished in single precision: nothing left to do
                while (from32 && s < n_starts && J.rec[s].status != GC_ST_PROMOTED) s = atomicAdd(next, 1ULL);
                sh.local[lane] = s;
                sh.born[lane] = T;
                sh.end[lane] = T + (s >= n_starts ? 0u : fixed ? J.fixed_sweeps[s] : (uint32_t)J.max_sweeps);
            }
            const uint64_t got = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(s >> 32), first) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((int)s, first);
            if (lane == 0) {
                const bool many = got + 8ULL * M * gridDim.x < n_starts;
                sh.spare = many;
                if (many) ahead = atomicAdd(next, 1ULL);
            }
        }
        __syncthreads();
        const bool free_place = lane < mmax && !((act >> lane) & 1u);
        const uint32_t got = (uint32_t)uniform((int)__ballot(free_place && sh.local[lane < M ? lane : 0] < n_starts));
        exhausted = (act | got) != all;
        spare = uniform(sh.spare) != 0;
        for (uint32_t left = got; left; left &= left - 1) {
            const int m = __builtin_ctz(left);
            // its start state, or the one promoted from single precision
            glb_ptr<const dbl2> in =
                as_global(reinterpret_cast<const dbl2 *>(J.states + uniform((uint64_t)sh.local[m]) * (uint64_t)V));
            for (int i = tid; i < V; i += B) {
                const dbl2 g = in[i];
                X[M * inv[i] + m] = C{(R)g.x, (R)g.y};
            }
        }
        act |= got;
        fresh |= got;
        __syncthreads();
    };

    // One start is left, and none to come (or one at a time, mmax = 1): it
    // goes on in the loop at the end.
    auto alone = [&]() __attribute__((always_inline)) {
        return LONE && every && (act & (act - 1)) == 0 && (mmax == 1 || (exhausted && !spare));
    };

    if (tid == 0) {
        sh.near = 0;
        sh.tally = RelaxTally{0, 0, 0};
    }
    refill();
    if constexpr (K == 2) {
        // a sweep: colour 0, barrier, colour 1, barrier.  The norm of the
        // sweep before it is complete after the first half and added up
        // beside the second; a start found to have stopped is put back by one
        // sweep from the values held in registers.
        while (act && !alone()) {
            const uint32_t pend = due();
            pass(std::integral_constant<int, 0>{}, act,
                 [&](auto mc, auto sc, const C *pf) __attribute__((always_inline)) {
                     constexpr int m = decltype(mc)::value, q = decltype(sc)::value;
                     const C g = *site(0, q, m);
                     const C sv = staple(0, q, m, pf);
                     old[0][m][q] = g;
                     *site(0, q, m) = team_update<RELAX, R>(g, sv, omega);
                     red[m * B + tid] = norm(q ? red[m * B + tid] : red1[m * B + tid], g, sv);
                 });
            __syncthreads();
            reduce(pend);
            pass(std::integral_constant<int, 1>{}, act,
                 [&](auto mc, auto sc, const C *pf) __attribute__((always_inline)) {
                     constexpr int m = decltype(mc)::value, q = decltype(sc)::value;
                     const C g = *site(1, q, m);
                     const C sv = staple(1, q, m, pf);
                     const C r = team_update<RELAX, R>(g, sv, omega);
                     old[1][m][q] = g;
                     *site(1, q, m) = r;
                     red1[m * B + tid] = norm(q ? red1[m * B + tid] : 0.0, r, sv);
                 });
            __syncthreads();
            const uint32_t near = (uint32_t)uniform((int)sh.near);
            const uint32_t fin = __builtin_expect(near != 0, 0) ? decide(near) : 0u;
            if (__builtin_expect(fin != 0, 0)) {
                each<M>([&](auto mc) __attribute__((always_inline)) {
                    constexpr int m = decltype(mc)::value;
                    if (!((fin >> m) & 1u)) return;
#pragma unroll
                    for (int q = 0; q < SPT; ++q) {
                        *site(0, q, m) = old[0][m][q];
                        *site(1, q, m) = old[1][m][q];
                    }
                });
                __syncthreads();
                finish(fin);
            }
            fresh = 0;
            ++T;
            if (__builtin_expect((!exhausted || spare) && act != all, 0)) refill();
        }
    } else {
        // a sweep: the norm of the last one with colour 0's staples, then
        // the colours in turn
        while (act && !alone()) {
            const uint32_t pend = due();
            pass(std::integral_constant<int, 0>{}, act,
                 [&](auto mc, auto sc, const C *pf) __attribute__((always_inline)) {
                     constexpr int m = decltype(mc)::value, q = decltype(sc)::value;
                     const C g = *site(0, q, m);
                     const C sv = staple(0, q, m, pf);
                     old[0][m][q] = team_update<RELAX, R>(g, sv, omega);
                     red[m * B + tid] = norm(red[m * B + tid], g, sv);
                 });
            if (pend) {
                each<K - 2>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int c = decltype(kc)::value + 1;
                    pass(std::integral_constant<int, c>{}, pend,
                         [&](auto mc, auto sc, const C *pf) __attribute__((always_inline)) {
                             constexpr int m = decltype(mc)::value, q = decltype(sc)::value;
                             const C g = *site(c, q, m);
                             red[m * B + tid] = norm(red[m * B + tid], g, staple(c, q, m, pf));
                         });
                });
                __syncthreads();
                reduce(pend);
                __syncthreads();
                const uint32_t near = (uint32_t)uniform((int)sh.near);
                if (__builtin_expect(near != 0, 0)) finish(decide(near));
            }
            each<M>([&](auto mc) __attribute__((always_inline)) {
                constexpr int m = decltype(mc)::value;
                if (!((act >> m) & 1u)) return;
#pragma unroll
                for (int q = 0; q < SPT; ++q) *site(0, q, m) = old[0][m][q];
            });
            __syncthreads();
            each<K - 1>([&](auto kc) __attribute__((always_inline)) {
                constexpr int c = decltype(kc)::value + 1;
                pass(std::integral_constant<int, c>{}, act,
                     [&](auto mc, auto sc, const C *pf) __attribute__((always_inline)) {
                         constexpr int m = decltype(mc)::value, q = decltype(sc)::value;
                         const C g = *site(c, q, m);
                         const C sv = staple(c, q, m, pf);
                         const C r = team_update<RELAX, R>(g, sv, omega);
                         *site(c, q, m) = r;
                         if (c == K - 1) red[m * B + tid] = norm(q ? red[m * B + tid] : 0.0, r, sv);
                     });
                __syncthreads();
            });
            fresh = 0;
            ++T;
            if (__builtin_expect((!exhausted || spare) && act != all, 0)) refill();
        }
    }

    // A start on its own: no other one fills its waits, so what counts is the
    // length of the chain through a sweep.  It moves to place 0 and runs Q
    // sweeps at a time; their norms are left in red and added up together, off
    // the chain, and a start found to have stopped among them is run again
    // from the copy in place 1 up to its last sweep.  A sweep takes 0.56 us on
    // 16^2 (0.93 in the loop above), 0.64 on 8^3 (0.99), 0.78 on 4^4 (1.15) and
    // 1.46 on 9^3 (1.98).  The links are loaded anew: held across both loops
    // they left the one above too few registers.
    if (!LONE || act == 0) {
        if (tid == 0) flush_tally(J, sh.tally);
        return;
    }
    load_links();
    __syncthreads();   // a start that ended in place 0 beside this one is written out
    constexpr int Q = (K == 2 ? 2 : 1) * M < 6 ? (K == 2 ? 2 : 1) * M : 6;
    while (act) {
        const int from = __builtin_ctz(act);
        double part = (K == 2 ? red1 : red)[from * B + tid];   // the norm's part from the last colour
        C own2[K == 2 ? 2 : 1][SPT];                           // two colours: the own sites' values
        each<K>([&](auto cc) __attribute__((always_inline)) {
            constexpr int c = decltype(cc)::value;
#pragma unroll
            for (int q = 0; q < SPT; ++q) {
                const C g = site(c, q, 0)[from];
                *site(c, q, 0) = g;
                if constexpr (K == 2) own2[c][q] = g;
            }
        });
        if (tid == 0 && from) {
            sh.local[0] = sh.local[from];
            sh.born[0] = sh.born[from];
            sh.end[0] = sh.end[from];
        }
        act = 1;
        bool first = fresh != 0;   // no sweep yet, no norm to look at
        fresh = 0;
        __syncthreads();
        const uint32_t end = (uint32_t)uniform((int)sh.end[0]);
        // one sweep; the norm of the state before it to red[q]
        auto sweep = [&](int q) __attribute__((always_inline)) {
            if constexpr (K == 2) {
                each<2>([&](auto cc) __attribute__((always_inline)) {
                    constexpr int c = decltype(cc)::value;
                    C sv[SPT];
#pragma unroll
                    for (int r = 0; r < SPT; ++r) sv[r] = staple(c, r, 0, nullptr);
                    double next_part = 0.0;
#pragma unroll
                    for (int r = 0; r < SPT; ++r) {
                        const C g = team_update<RELAX, R>(own2[c][r], sv[r], omega);
                        if (c == 0) part = norm(part, own2[c][r], sv[r]);
                        else next_part = norm(next_part, g, sv[r]);
                        own2[c][r] = g;
                        *site(c, r, 0) = g;
                    }
                    if (c == 0) red[q * B + tid] = part;
                    else part = next_part;
                    __syncthreads();
                });
            } else {
                C g0[SPT];
#pragma unroll
                for (int r = 0; r < SPT; ++r) {
                    const C g = *site(0, r, 0);
                    const C sv = staple(0, r, 0, nullptr);
                    part = norm(part, g, sv);
                    g0[r] = team_update<RELAX, R>(g, sv, omega);
                }
                each<K - 2>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int c = decltype(kc)::value + 1;
#pragma unroll
                    for (int r = 0; r < SPT; ++r) {
                        const C g = *site(c, r, 0);
                        part = norm(part, g, staple(c, r, 0, nullptr));
                    }
                });
                red[q * B + tid] = part;
                __syncthreads();
#pragma unroll
                for (int r = 0; r < SPT; ++r) *site(0, r, 0) = g0[r];
                __syncthreads();
                each<K - 1>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int c = decltype(kc)::value + 1;
                    part = 0.0;
#pragma unroll
                    for (int r = 0; r < SPT; ++r) {
                        const C sv = staple(c, r, 0, nullptr);
                        const C g = team_update<RELAX, R>(*site(c, r, 0), sv, omega);
                        *site(c, r, 0) = g;
                        if (c == K - 1) part = norm(part, g, sv);
                    }
                    __syncthreads();
                });
            }
        };
        for (;;) {
            // the own sites' values to place 1
            each<K>([&](auto cc) __attribute__((always_inline)) {
                constexpr int c = decltype(cc)::value;
#pragma unroll
                for (int q = 0; q < SPT; ++q) site(c, q, 0)[1] = *site(c, q, 0);
            });
            for (int q = 0; q < Q; ++q) sweep(q);
            // norm q to sh.lone[q], the additions of reduce
            for (int q = wave; q < Q; q += waves) {
                double x[MAXW];
#pragma unroll
                for (int w = 0; w < MAXW; ++w) x[w] = red[q * B + 64 * min(w, waves - 1) + lane];
                double v = x[0];
#pragma unroll
                for (int w = 1; w < MAXW; ++w) {
                    const double y = w < waves ? x[w] : 0.0;
                    v = MAXABS ? fmax(v, y) : v + y;
                }
                v = MAXABS ? wave_max(v) : wave_sum(v);
                if (lane == 0) sh.lone[q] = v;
            }
            __syncthreads();
            // the first sweep after which the start stops, lane q looks at q
            const double v = sh.lone[lane < Q ? lane : 0];
            const double Dn = MAXABS ? v : v / (double)V;
            const bool bad = !(Dn == Dn), conv = Dn < eps;
            const uint64_t stops = __ballot(lane < Q && (lane > 0 || !first) && (bad || conv || T + (uint32_t)lane == end));
            first = false;
            if (stops == 0) {
                T += Q;
                continue;
            }
            const int n = __builtin_ctzll(stops);
            if (lane == n) {
                sh.D[0] = Dn;
                sh.status[0] = bad ? GC_ST_BADNUM : conv ? GC_ST_CONVERGED : GC_ST_NONCONVERGED;
                sh.sweeps[0] = T + (uint32_t)n - sh.born[0];
            }
            each<K>([&](auto cc) __attribute__((always_inline)) {
                constexpr int c = decltype(cc)::value;
#pragma unroll
                for (int q = 0; q < SPT; ++q) {
                    const C g = site(c, q, 0)[1];
                    *site(c, q, 0) = g;
                    if constexpr (K == 2) own2[c][q] = g;
                }
            });
            __syncthreads();
            for (int q = 0; q < n; ++q) sweep(0);
            T += (uint32_t)n;
            break;
        }
        finish(1u);
        if (!exhausted || spare) refill();
    }
    if (tid == 0) flush_tally(J, sh.tally);
}

// Workgroups move from job to job of the launch as their starts run out.
template <int D, int K, int CLS, typename R, int RM>
__global__ __launch_bounds__(64 * gc_team_class(D, K, CLS).maxw, gc_team_class(D, K, CLS).minw) void team_kernel(
    const GcJobDev *__restrict__ jobs, int n_jobs, unsigned long long *job_next, int mmax)
{
    constexpr GcTeamClass TC = gc_team_class(D, K, CLS);
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int cur_job;
    __shared__ TeamShared<TC.m> sh;
    static_assert(sizeof sh + sizeof cur_job <= 1024, "beside the 159 KiB that gc_team_shape allows");
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
        team_job<D, K, TC.spt, TC.m, TC.maxw, TC.pf, TC.lone || sizeof(R) == 4, R, (RM & 1) != 0, (RM & 2) != 0>(
            jobs[jn], &job_next[jn], mmax, smem, sh);
        __syncthreads();
        j0 = jn;
    }
}

}  // namespace
