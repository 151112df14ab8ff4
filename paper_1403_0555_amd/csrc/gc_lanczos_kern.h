// FP filter in the line-segment layout (the fast filter kernel), templated
// on the lattice dimension and instantiated per dimension in
// gc_lanczos1.hip .. gc_lanczos4.hip.
#pragma once

#include "gc_filter.h"

namespace {

// The Lanczos tridiagonal in LDS, row j as (alpha_j, beta_{j-1}^2), followed
// by kTriPad rows past the last.
typedef __attribute__((address_space(3))) const dbl2 lds_cdbl2;
constexpr int kTriPad = GC_TRI_PAD;

// p_k(x) = det(T_k - x) up to a positive smooth factor, as f 2^e, and whether
// an eigenvalue lies below x: the Sturm sequence of sturm_count (gc_filter.h)
// has a sign change.  Rows come four at a time, loaded one block ahead; rows
// past the last stand for alpha = 64 > x, beta = 0 and keep every sign.  The
// pair is rescaled after eight rows: |alpha - x| < 2^7 and beta^2 < 2^10
// leave it in range.  A row takes three double-precision and two integer
// instructions on the wavefront, 20 cycles (64 with the rows loaded where
// they are used, signs counted and a rescaling every four rows).
struct SturmValue {
    double f;
    int e;
    bool below;
};
__device__ __forceinline__ SturmValue sturm_value(lds_cdbl2 *tri, int k, double x)
{
    double p0 = 0.0, p1 = 1.0;
    uint32_t signs = 0;
    int e = 0;
    auto rows = [&](const dbl2 (&row)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double p2 = fma(row[u].x - x, p1, -row[u].y * p0);
            signs |= (uint32_t)(((uint64_t)__double_as_longlong(p2) ^ (uint64_t)__double_as_longlong(p1)) >> 32);
            p0 = p1;
            p1 = p2;
        }
    };
    dbl2 ra[4], rb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) ra[u] = tri[u];
    for (int j = 0; j < k; j += 8) {
#pragma unroll
        for (int u = 0; u < 4; ++u) rb[u] = tri[j + 4 + u];
        rows(ra);
        const int jn = min(j + 8, k);   // the rows past the last where no block follows
#pragma unroll
        for (int u = 0; u < 4; ++u) ra[u] = tri[jn + u];
        rows(rb);
        int q;
        (void)frexp(p1, &q);
        p0 = ldexp(p0, -q);
        p1 = ldexp(p1, -q);
        e += q;
    }
    return {p1, e, (signs >> 31) != 0};
}

__device__ __forceinline__ double lane_value(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// a / b to about 2^-45: the estimate refined once.
__device__ __forceinline__ double quick_div(double a, double b)
{
    const double r = __builtin_amdgcn_rcp(b);
    return a * fma(r, fma(-b, r, 1.0), r);
}

// The lowest root of p_k by inverse cubic interpolation from four
// neighbouring lanes' values, lane l's point at u = l: the root in these
// units and, as its uncertainty, how far the quadratic ones are from it.
__device__ __forceinline__ double root_estimate(const SturmValue &s, int first, double &err)
{
    const int b = min(max(first - 2, 0), 60);
    const int eb = __builtin_amdgcn_readlane(s.e, b + 1);
    const double g = ldexp(s.f, max(min(s.e - eb, 600), -600));
    const double f0 = lane_value(g, b), f1 = lane_value(g, b + 1), f2 = lane_value(g, b + 2), f3 = lane_value(g, b + 3);
    // u - b = 0, 1, 2, 3
    const double p01 = quick_div(f0, f0 - f1);
    const double p12 = quick_div(2.0 * f1 - f2, f1 - f2);
    const double p23 = quick_div(3.0 * f2 - 2.0 * f3, f2 - f3);
    const double p012 = quick_div(f0 * p12 - f2 * p01, f0 - f2);
    const double p123 = quick_div(f1 * p23 - f3 * p12, f1 - f3);
    const double p = quick_div(f0 * p123 - f3 * p012, f0 - f3);
    err = fmax(fabs(p - p012), fabs(p - p123));
    return (double)b + p;
}

// ritz_min and tridiag_min_eig of gc_filter.h on one wavefront, the same
// brackets bit for bit.  A round of 64 points takes a Sturm sequence each;
// the values they leave give the root far beyond the next bracket
// (root_estimate), so the brackets of the rounds to come are worked out from
// the estimate and one more round, with their ends on its lanes, shows which
// of them hold.  A bracket whose ends have no eigenvalue below, and one, is
// the one that the 64 points of its round would have given.  Two to three
// rounds in place of four to six.
__device__ double ritz_lines(lds_cdbl2 *tri, int k, double glo, double ghi, double prev, double prev_step,
                             double tol_rel, bool final, double &hi_out)
{
    constexpr int B = 64;
    const int lane = (int)(threadIdx.x & 63);
    double lo = glo - 1e-12 * (1.0 + fabs(glo));
    double hi = ghi + 1e-12 * (1.0 + fabs(ghi));
    SturmValue s = {0.0, 0, false};
    int first = -1;           // of the last round, -1: no values to go by
    double u0 = 0.0, du = 0.0;   // its points: u0 + du l
    if (prev < hi) {
        const double top = prev + 1e-12 * (1.0 + fabs(prev));
        const double bot = top - fmax(4.0 * prev_step, 1e-9 * (1.0 + fabs(prev)));
        if (bot > lo) {
            const double step = (top - bot) / (double)(B - 1);
            const double x = (lane == B - 1) ? top : bot + step * (double)lane;
            s = sturm_value(tri, k, x);
            const uint64_t m = __ballot(s.below);
            first = m ? __builtin_ctzll(m) : B;
            if (first > 0 && first < B) {
                lo = bot + step * (double)(first - 1);
                hi = (first == B - 1) ? top : bot + step * (double)first;
                u0 = bot;
                du = step;
            } else {
                if (first == 0) hi = bot;   // below the window: bot bounds it above
                first = -1;
            }
        } else if (sturm_value(tri, k, top).below) {
            hi = top;
        }
    }
    const double width = final ? 1e-15 : 1e-2 * tol_rel;
    // the search is over: the bracket is narrow enough, or, unless final, the
    // convergence test fails whatever the remaining digits are
    auto over = [&](double l, double h) __attribute__((always_inline)) {
        if (h - l <= width * fmax(1.0, fabs(h))) return true;
        if (!final) {
            const double gap = prev - h, scale = fmax(1.0, fabs(h));
            const bool fails = gap > 1e6 * tol_rel * scale;
            const double need = (prev < INFINITY) ? 0.05 * gap : 1e-4 * scale;
            if (fails && h - l <= need) return true;
        }
        return false;
    };
    int round = 0;
    while (round < 24 && !over(lo, hi)) {
        if (first >= 0 && !final) {
            double err;
            const double u = root_estimate(s, first, err);
            const double r = fma(du, u, u0), unsure = 4.0 * du * err;
            // the brackets of the rounds to come, one per pair of lanes
            double pl = lo, ph = hi, x = lo;
            int n = 0;
            while (n < 16 && round + n < 24 && !over(pl, ph)) {
                const double step = (ph - pl) / (double)(B + 1);
                const double q = (r - pl) / step;
                // the estimate has to tell the round's points apart
                if (!(unsure < 0.25 * step) || !(q >= -1.0 && q <= (double)(B + 2))) break;
                const int f = min(max((int)floor(q), 0), B);
                const double nlo = (f == 0) ? pl : pl + step * (double)f;
                const double nhi = (f == B) ? ph : pl + step * (double)(f + 1);
                pl = nlo;
                ph = nhi;
                x = (lane == 2 * n) ? pl : (lane == 2 * n + 1) ? ph : x;
                ++n;
            }
            if (n > 0) {
                const uint64_t m = __ballot(sturm_value(tri, k, x).below);
                // pairs (0, 1) from the first on
                int ok = 0;
                while (ok < n && ((m >> (2 * ok)) & 3ull) == 2ull) ++ok;
                // replay the brackets that hold
                for (int i = 0; i < ok; ++i) {
                    lo = lane_value(x, 2 * i);
                    hi = lane_value(x, 2 * i + 1);
                }
                round += ok;
                first = -1;
                if (ok == n) continue;
            }
            if (round >= 24 || over(lo, hi)) break;
        }
        const double step = (hi - lo) / (double)(B + 1);
        const double x = lo + step * (double)(lane + 1);
        s = sturm_value(tri, k, x);
        const uint64_t m = __ballot(s.below);
        first = m ? __builtin_ctzll(m) : B;
        const double nlo = (first == 0) ? lo : lo + step * (double)first;
        const double nhi = (first == B) ? hi : lo + step * (double)(first + 1);
        u0 = lo + step;
        du = step;
        lo = nlo;
        hi = nhi;
        ++round;
    }
    hi_out = hi;
    return 0.5 * (lo + hi);
}

// The Ritz value of a check, computed by the first wavefront alone and
// handed to the others through LDS.  The workgroup synchronises before (the
// tridiagonal is complete in LDS) and after.
template <int B>
__device__ double ritz_wave0(lds_ptr<dbl2> tri, int k, double glo, double ghi, double prev, double prev_step,
                             bool final, double &hi_out, double *share)
{
    if (B > 64) __syncthreads();
    else wave_sync();
    double theta = 0.0, hi = 0.0;
    if (B == 64 || threadIdx.x < 64) {
        if ((threadIdx.x & 63) < kTriPad) tri[k + (int)(threadIdx.x & 63)] = dbl2{64.0, 0.0};
        wave_sync();
        theta = ritz_lines((lds_cdbl2 *)tri, k, glo, ghi, prev, prev_step, kRitzTol, final, hi);
        if (B > 64 && threadIdx.x == 0) {
            share[0] = theta;
            share[1] = hi;
        }
    }
    if (B > 64) {
        __syncthreads();
        theta = share[0];
        hi = share[1];
    }
    hi_out = hi;
    return theta;
}

// Four sums over the workgroup, each with the additions of wg_sum_n
// (gc_filter.h) in the same order.  Two steps inside a quad halve the values
// a lane carries (it passes on the ones it gives up), so the four steps that
// remain move one value and not four: 35 vector instructions against 80.
// Lane l ends with the sum of class (l & 3), reversed in odd quads, where the
// mirror steps then find the same class.
template <int B> __device__ __forceinline__ void wg_sum4(double (&v)[4], double *red, int &ph)
{
    const int lane = (int)(threadIdx.x & 63);
    const bool c1 = ((lane ^ (lane >> 2)) & 1) != 0, c2 = (((lane >> 1) ^ (lane >> 2)) & 1) != 0;
    double x[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const double keep = c1 ? v[2 * n + 1] : v[2 * n], give = c1 ? v[2 * n] : v[2 * n + 1];
        x[n] = keep + dpp64<kDppQuadSwap1>(give);
    }
    const double keep = c2 ? x[1] : x[0], give = c2 ? x[0] : x[1];
    double y = keep + dpp64<kDppQuadSwap2>(give);
    y += dpp64<kDppHalfMirror>(y);
    y += dpp64<kDppRowMirror>(y);
    RowPair p = row_pair<16>(y);
    y = p.lo + p.hi;
    p = row_pair<32>(y);
    y = p.lo + p.hi;
    if (B > 64) {
        // lane l adds up the wavefronts' sums of class (l & 3)
        constexpr int W = B / 64;
        double *r = red + ph * (4 * W);
        ph ^= 1;
        if (lane < 4) r[lane * W + (threadIdx.x >> 6)] = y;
        __syncthreads();
        const double *rl = r + (lane & 3) * W;
        y = rl[0];
#pragma unroll
        for (int w = 1; w < W; ++w) y += rl[w];
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) v[n] = lane_value(y, n);
}

// FP filter in the line-segment layout, one workgroup of B threads per copy
// of the compacted tables (at the copy's representative start): thread t
// owns S consecutive sites along direction 0 (x_0 runs fastest, so they are
// consecutive site indices), segment t % (N_0/S) of line t / (N_0/S).  The
// Lanczos vector u of the own sites, q_{j-1} and M u stay in registers, and
// so do the direction-0 link weights; direction-0 neighbours inside the
// segment are the thread's own entries.  LDS holds u for the other
// threads, the forward link weights of directions 1..d-1 (and of direction
// 0 when a line has several segments), S P doubles each, and the
// tridiagonal.  LDS arrays are segment-major with a compile-time stride P
// (B, or 7B/8 when the launch's T = V/S threads fit in it), two sites of a
// thread side by side: sites k and k + 1 (k even) of thread t's segment sit
// at k P + 2 t, the last of an odd segment at (S - 1) P + t.  A wavefront
// touches consecutive pairs, one 16-byte access each (217 bytes per clock of
// a CU against 118 in 8-byte accesses), a neighbour in direction mu >= 1
// (the same k of another segment) sits at a constant thread offset, and every
// site's address is one of 2 d per-thread bases plus a compile-time offset.
// FORM bit 0: the segments are whole lines (S == N0); bit 1: P = 7B/8.  The
// iteration is post_kernel's: one reduction per iteration, the same formulas
// per site.
//
// Per iteration LDS moves 4 (d - 1) + 1 values per site, 50 KB on 6^4, and the
// reduction's and the checks' latency comes on top; several workgroups per
// CU hide it, as many as registers and LDS allow.  Copies filtered, before
// and after pairs, wg_sum4 and ritz_lines: 100000 on 6^4 38.8 -> 31.0 ms,
// 100000 on 10^3 25.9 -> 21.1, 10000 on 9^3 3.08 -> 2.08, 4000 on 12^3
// 5.07 -> 3.64, 2000 on 6^3 x 8 2.53 -> 1.85, 4000 on 32^2 2.06 -> 1.29, 20000 on 16^2
// 1.39 -> 1.04.

// Wavefronts per SIMD the filter is compiled for: five values a site in
// registers (10 S), and addresses, scalars and loads in flight, about
// 98 + 2 D more.  Some 15 registers over the limit of 512 / waves are spilled
// outside the iteration and cost less than the wavefront: 10000 copies on 9^3
// (S = 3) take 2.08 ms with four wavefronts and 2.32 with three, 36000 on
// 8^3 (S = 8) 3.03 with three and 3.12 with two.  512 threads are two
// wavefronts on each SIMD: two or four (3 x 21 x 21: 3.87 and 2.54 ms).
constexpr int lanczos_waves(int B, int S, int D)
{
    const int regs = 10 * S + 2 * D + 98;
    return regs <= 142 ? 4 : regs <= 186 && B < 512 ? 3 : 2;
}

template <int B, int S, int D, int FORM>
__global__ __launch_bounds__(B, lanczos_waves(B, S, D)) void lanczos_kernel(const GcJobDev *__restrict__ jobs, int n_jobs,
                                                    unsigned long long *next)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2 * 4 * (B / 64)];
    __shared__ double ritz[2];
    __shared__ unsigned long long claim;
    int rph = 0;   // half of the reduction scratch in use
    // copies filtered and not yet in their job's counter; copies come in job
    // order
    uint32_t runs = 0;
    int runs_job = 0;
    for (;;) {
        const int tid = (int)threadIdx.x + opaque_zero();
        if (tid == 0) claim = atomicAdd(next, 1ULL);
        __syncthreads();
        const uint64_t s = uniform((uint64_t)claim);
        __syncthreads();
        int jn;
        uint64_t c;
        copy_item(jobs, n_jobs, s, jn, c);
        jn = uniform(jn);
        if (jn != runs_job) {
            if (tid == 0 && runs) atomicAdd(&jobs[runs_job].cnt->lanczos_runs, (unsigned long long)runs);
            runs = 0;
            runs_job = jn;
        }
        if (jn < 0) break;
        const GcJobDev &J = jobs[jn];
        const GcOrbitDev &O = J.orb;
        const int V = O.V, N0 = O.ext[0];
        constexpr int d = D;   // the jobs of a launch share the dimension
        const uint64_t local = J.copies[c].rep_start - J.first_start;
        const int nseg = N0 / S;
        const bool act = tid < V / S;
        const int line = act ? tid / nseg : 0, o = act ? (tid % nseg) * S : 0;
        const int i0 = line * N0 + o;
        constexpr bool whole = (FORM & 1) != 0;   // the segment is a whole line (S == N0)
        constexpr int P = (FORM & 2) ? 7 * B / 8 : B;   // stride of the segment-major arrays (>= V/S)
        const int nw = whole ? d - 1 : d;   // weight arrays in LDS
        const int w0off = whole ? -1 : 0;   // LDS array of direction mu: mu + w0off
        constexpr int A = S * P;            // doubles per LDS array
        // place of the k-th site of thread t's segment in an LDS array
        auto at = [&](int k, int t) __attribute__((always_inline)) {
            return k < 2 * (S / 2) ? 2 * ((k >> 1) * P + t) + (k & 1) : k * P + t;
        };
        lds_ptr<double> u = as_lds(reinterpret_cast<double *>(smem));
        lds_ptr<double> wl = u + A;
        const int lmax = min(min(J.lanczos_max, GC_LMAX), V);
        lds_ptr<dbl2> tri = (lds_ptr<dbl2>)(wl + (size_t)nw * A);

        // own link weights w = Re(conj(g_i) U_{i,mu} g_{i+mu}) from the
        // representative's state in global memory: direction 0 into
        // registers, the others into LDS
        glb_ptr<const dbl2> src = as_global(reinterpret_cast<const dbl2 *>(J.states + local * (uint64_t)V));
        glb_ptr<const dbl2> Ug = as_global(reinterpret_cast<const dbl2 *>(O.U64));
        double w0[S];
        // thread offsets of the neighbours in directions >= 1 (the same for
        // every own site: site offsets, multiples of N0, divided by S)
        int df[GC_MAXD], db[GC_MAXD];
#pragma unroll
        for (int mu = 0; mu < GC_MAXD; ++mu) {
            df[mu] = 0;
            db[mu] = 0;
            if (act && mu > 0 && mu < d) {
                df[mu] = ((int)O.nbr[mu * V + i0] - i0) / S;
                db[mu] = ((int)O.nbr[(d + mu) * V + i0] - i0) / S;
            }
        }
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int i = i0 + k;
            w0[k] = 0.0;
            if (act) {
                const dbl2 gi = src[i];
#pragma unroll
                for (int mu = 0; mu < GC_MAXD; ++mu) {
                    if (mu < d) {
                        const dbl2 gf = src[O.nbr[mu * V + i]];
                        const dbl2 uu = Ug[mu * V + i];
                        const double tr = uu.x * gf.x - uu.y * gf.y, ti = uu.x * gf.y + uu.y * gf.x;
                        const double ur = gi.x * tr + gi.y * ti;
                        if (mu == 0) w0[k] = ur;
                        if (mu + w0off >= 0) wl[(mu + w0off) * A + at(k, tid)] = ur;
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        double uo[S], qp[S], mv[S];
        double sums[1] = {0.0};
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int i = i0 + k;
            qp[k] = 0.0;
            uo[k] = 0.0;
            mv[k] = 0.0;
            if (act) {
                const double x = (double)(mix64((uint64_t)i + 0x5851F42D4C957F2DULL) >> 11) * 0x1.0p-53 - 0.5;
                uo[k] = x;
                sums[0] += x;
            }
        }
        wg_sum_n<B, 1>(sums, red, rph);
        const double mean = sums[0] / (double)V;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            if (act) {
                uo[k] -= mean;
                u[at(k, tid)] = uo[k];
            }
        }
        const double sigma = 4.0 * d + 1.0;
        const double sigma_v = sigma / (double)V;   // the weight of the projector on the constant vector
        double theta = INFINITY, theta_old = INFINITY, theta_step = 1.0;
        double rows_lo = INFINITY, rows_hi = -INFINITY;   // Gershgorin bounds of the complete rows
        double a_prev = 0.0, b_prev2 = 0.0;                // alpha_{j-1}, beta_{j-2}
        int next_check = kFirstCheck;                      // iteration count of the next Ritz check
        int it = 0;
        bool conv = false;
        // the neighbours across the ends of a segment that is not a whole
        // line: the first site of the next segment, the last of the previous
        const int ia = at(0, line * nseg + ((o + S) % N0) / S);
        const int ib = at(S - 1, line * nseg + ((o + N0 - 1) % N0) / S);
        // byte offsets of pair 0 in LDS: the thread's, and its neighbours'
        lds_ptr<unsigned char> u8 = (lds_ptr<unsigned char>)u;
        const uint32_t t16 = 16u * (uint32_t)tid;
        uint32_t f16[GC_MAXD], b16[GC_MAXD];
#pragma unroll
        for (int mu = 0; mu < GC_MAXD; ++mu) {
            f16[mu] = 16u * (uint32_t)(tid + df[mu]);
            b16[mu] = 16u * (uint32_t)(tid + db[mu]);
        }
        // the diagonal of M at the own sites, the sum of their 2d link
        // weights, once per copy (M u)_i = diag_i u_i - sum_nb w u_nb
        if (B > 64) __syncthreads();   // the weights complete in LDS
        else wave_sync();
        double dg[S];
        {
            const double wbe0 = whole ? w0[S - 1] : wl[ib];
            const int ta = act ? tid : 0;   // threads past the stride P would read past the arrays
#pragma unroll
            for (int k = 0; k < S; ++k) {
                double a = w0[k] + ((k > 0) ? w0[k - 1] : wbe0);
#pragma unroll
                for (int mu = 1; mu < GC_MAXD; ++mu)
                    if (mu < d) {
                        lds_ptr<const double> wm = wl + (mu + w0off) * A;
                        a += wm[at(k, ta)] + wm[at(k, ta + db[mu])];
                    }
                dg[k] = act ? a : 0.0;
            }
        }
        for (it = 0; it < lmax; ++it) {
            if (B > 64) __syncthreads();   // u and the weights complete in LDS
            else wave_sync();
            double s4[4] = {0.0, 0.0, 0.0, 0.0};
            if (act) {
                double ua, ub, wbe;
                if constexpr (whole) {
                    ua = uo[0];
                    ub = uo[S - 1];
                    wbe = w0[S - 1];
                } else {
                    ua = u[ia];
                    ub = u[ib];
                    wbe = wl[ib];
                }
                // two sites at a time, their values side by side in LDS
#pragma unroll
                for (int k0 = 0; k0 < S; k0 += 2) {
                    const int n = k0 + 1 < S ? 2 : 1;
                    double m[2];
#pragma unroll
                    for (int h = 0; h < n; ++h) {
                        // direction 0: neighbours and weights of the own segment
                        const int k = k0 + h;
                        m[h] = dg[k] * uo[k];
                        m[h] = fma(-w0[k], (k + 1 < S) ? uo[k + 1] : ua, m[h]);
                        m[h] = fma(-((k > 0) ? w0[k - 1] : wbe), (k > 0) ? uo[k - 1] : ub, m[h]);
                    }
#pragma unroll
                    for (int mu = 1; mu < GC_MAXD; ++mu)
                        if (mu < d) {
                            // the pair's place is a constant from the
                            // thread's; a last single site's likewise from
                            // half of it
                            const uint32_t w8 = 8u * (uint32_t)((1 + mu + w0off) * A);
                            if (n == 2) {
                                const uint32_t kb = 16u * (uint32_t)((k0 >> 1) * P);
                                const dbl2 wf = *(lds_ptr<const dbl2>)(u8 + t16 + (w8 + kb));
                                const dbl2 uf = *(lds_ptr<const dbl2>)(u8 + f16[mu] + kb);
                                const dbl2 wb = *(lds_ptr<const dbl2>)(u8 + b16[mu] + (w8 + kb));
                                const dbl2 ub2 = *(lds_ptr<const dbl2>)(u8 + b16[mu] + kb);
                                m[0] = fma(-wf.x, uf.x, m[0]);
                                m[1] = fma(-wf.y, uf.y, m[1]);
                                m[0] = fma(-wb.x, ub2.x, m[0]);
                                m[1] = fma(-wb.y, ub2.y, m[1]);
                            } else {
                                const uint32_t kb = 8u * (uint32_t)(k0 * P);
                                const double wf = *(lds_ptr<const double>)(u8 + (t16 >> 1) + (w8 + kb));
                                const double uf = *(lds_ptr<const double>)(u8 + (f16[mu] >> 1) + kb);
                                const double wb = *(lds_ptr<const double>)(u8 + (b16[mu] >> 1) + (w8 + kb));
                                const double ub2 = *(lds_ptr<const double>)(u8 + (b16[mu] >> 1) + kb);
                                m[0] = fma(-wf, uf, m[0]);
                                m[0] = fma(-wb, ub2, m[0]);
                            }
                        }
#pragma unroll
                    for (int h = 0; h < n; ++h) {
                        const int k = k0 + h;
                        mv[k] = m[h];
                        s4[0] += uo[k] * uo[k];
                        s4[1] += uo[k] * m[h];
                        s4[2] += uo[k];
                        s4[3] += uo[k] * qp[k];
                    }
                    // bounds the loads in flight
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            wg_sum4<B>(s4, red, rph);
            // 1/|u| from the reciprocal square root, no division on the
            // iteration's dependency chain (a vanishing |u| gives bt = 0)
            const double inv = rsq(fmax(s4[0], 1e-300));
            const double bt = s4[0] * inv;
            const double bp = it > 0 ? bt : 0.0;      // beta_{j-1} (the start vector's norm is not in T)
            if (it > 0) {
                rows_lo = fmin(rows_lo, a_prev - b_prev2 - bt);
                rows_hi = fmax(rows_hi, a_prev + b_prev2 + bt);
                if (bt <= 1e-13 * sigma) {
                    // the Krylov space is exhausted: T of it rows is exact
                    double theta_hi;
                    theta = ritz_wave0<B>(tri, it, rows_lo, rows_hi, theta_old, theta_step, true, theta_hi, ritz);
                    conv = true;
                    break;
                }
            }
            const double sq = s4[2] * inv;
            const double shift = sigma_v * sq;
            const double a_j = s4[1] * inv * inv + shift * sq - bp * (s4[3] * inv);
            if (tid == 0) tri[it] = dbl2{a_j, it > 0 ? s4[0] : 0.0};
            if (act) {
#pragma unroll
                for (int k = 0; k < S; ++k) {
                    const double q = uo[k] * inv;
                    const double r = mv[k] * inv + shift - bp * qp[k] - a_j * q;
                    qp[k] = q;
                    uo[k] = r;
                }
#pragma unroll
                for (int k = 0; k < S; k += 2) {
                    if (k + 1 < S) *(lds_ptr<dbl2>)(u8 + t16 + 16u * (uint32_t)((k >> 1) * P)) = dbl2{uo[k], uo[k + 1]};
                    else *(lds_ptr<double>)(u8 + (t16 >> 1) + 8u * (uint32_t)(k * P)) = uo[k];
                }
            }
            if (it + 1 >= next_check || it + 1 == lmax) {
                const bool final = it + 1 == lmax;
                double theta_hi;
                theta = ritz_wave0<B>(tri, it + 1, fmin(rows_lo, a_j - bp), fmax(rows_hi, a_j + bp), theta_old,
                                      theta_step, final, theta_hi, ritz);
                const double tol = kRitzTol * fmax(1.0, fabs(theta));
                const double change = theta_old - theta;
                if (fabs(change) <= tol) {
                    conv = true;
                    ++it;
                    break;
                }
                const int gap = check_gap(change, tol);
                next_check = it + 1 + gap;
                if (theta_old < INFINITY) theta_step = change;
                theta_old = theta_hi;
            }
            b_prev2 = bp;
            a_prev = a_j;
        }
        uint32_t flags = region_flags(theta, J.lambda_tol);
        if (!conv) flags |= GC_F_LANCZOS_CAP;
        if (tid == 0) {
            write_filter(J, c, local, theta, flags, (uint32_t)it);
            if (++runs == 16) {
                atomicAdd(&J.cnt->lanczos_runs, 16ULL);
                runs = 0;
            }
        }
        __syncthreads();
    }
}

}  // namespace

// Entry points of one lattice dimension D (gc_lanczosD.hip): occupancy and
// launch of lanczos_kernel<B, S, D, FORM> for the shapes gc_lanczos_shape
// and gc_lanczos_form pick.
#define GC_LANCZOS_F(FN, B, S, D, ...)                                                                    \
    switch (form) {                                                                                       \
    case 0: return FN<B, S, D, 0>(__VA_ARGS__);                                                           \
    case 1: return FN<B, S, D, 1>(__VA_ARGS__);                                                           \
    case 2: return FN<B, S, D, 2>(__VA_ARGS__);                                                           \
    case 3: return FN<B, S, D, 3>(__VA_ARGS__);                                                           \
    default: return hipErrorInvalidValue;                                                                 \
    }
#define GC_LANCZOS_SEG(FN, B, D, ...)                                                                     \
    switch (seg) {                                                                                        \
    case 1: GC_LANCZOS_F(FN, B, 1, D, __VA_ARGS__)                                                        \
    case 2: GC_LANCZOS_F(FN, B, 2, D, __VA_ARGS__)                                                        \
    case 3: GC_LANCZOS_F(FN, B, 3, D, __VA_ARGS__)                                                        \
    case 4: GC_LANCZOS_F(FN, B, 4, D, __VA_ARGS__)                                                        \
    case 5: GC_LANCZOS_F(FN, B, 5, D, __VA_ARGS__)                                                        \
    case 6: GC_LANCZOS_F(FN, B, 6, D, __VA_ARGS__)                                                        \
    case 7: GC_LANCZOS_F(FN, B, 7, D, __VA_ARGS__)                                                        \
    case 8: GC_LANCZOS_F(FN, B, 8, D, __VA_ARGS__)                                                        \
    case 10: GC_LANCZOS_F(FN, B, 10, D, __VA_ARGS__)                                                      \
    default: return hipErrorInvalidValue;                                                                 \
    }
#define GC_LANCZOS_DISPATCH(FN, D, ...)                                                                   \
    switch (block) {                                                                                      \
    case 64: GC_LANCZOS_SEG(FN, 64, D, __VA_ARGS__)                                                       \
    case 128: GC_LANCZOS_SEG(FN, 128, D, __VA_ARGS__)                                                     \
    case 256: GC_LANCZOS_SEG(FN, 256, D, __VA_ARGS__)                                                     \
    case 512: GC_LANCZOS_SEG(FN, 512, D, __VA_ARGS__)                                                     \
    default: return hipErrorInvalidValue;                                                                 \
    }

template <int B, int S, int D, int FORM>
static hipError_t lanczos_occ_t(size_t lds, int *per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, lanczos_kernel<B, S, D, FORM>, B, lds);
}

template <int B, int S, int D, int FORM>
static hipError_t lanczos_launch_t(const GcJobDev *jobs, int n_jobs, unsigned long long *next, int grid, size_t lds,
                                   hipStream_t s)
{
    hipLaunchKernelGGL((lanczos_kernel<B, S, D, FORM>), dim3(grid), dim3(B), lds, s, jobs, n_jobs, next);
    return hipGetLastError();
}

// form: gc_lanczos_form's value, the same for every job of the launch
#define GC_LANCZOS_DEFINE_DIM(D)                                                                          \
    hipError_t gc_lanczos_occupancy_d##D(int block, int seg, int form, size_t lds_bytes,                  \
                                         int *blocks_per_cu)                                              \
    {                                                                                                     \
        GC_LANCZOS_DISPATCH(lanczos_occ_t, D, lds_bytes, blocks_per_cu)                                   \
    }                                                                                                     \
    hipError_t gc_launch_lanczos_d##D(int block, int seg, int form, const GcJobDev *jobs, int n_jobs,     \
                                      unsigned long long *next, int grid, size_t lds_bytes, hipStream_t s)  \
    {                                                                                                     \
        GC_LANCZOS_DISPATCH(lanczos_launch_t, D, jobs, n_jobs, next, grid, lds_bytes, s)                  \
    }
