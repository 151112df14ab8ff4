// Maximal Abelian reduction of an SU(2) configuration (Sec. I): the Landau
// functional of eq. (1) is stated for SU(N_c), and the Neuberger problem of
// SU(N_c) lies in its maximal Abelian subgroup U(1)^{N_c - 1}, the coset part
// being free of it.  The configuration is gauge-fixed on the coset SU(2)/U(1)
// to the maximal Abelian gauge -- R = sum_{x,mu} 1/2 Tr(s3 U' s3 U'^dagger),
// U' = g_x U_{x,mu} g_{x+mu}^dagger, maximised site by site, colour by
// colour -- and the diagonal phases of U' are the compact U(1) orbit whose
// Landau-gauge copies the rest of the library enumerates.
//
// Quaternions q = (q0, q1, q2, q3) stand for q0 + i (q1 s1 + q2 s2 + q3 s3).
// R depends on g_x only through the axis n_x, n . s = g_x^dagger s3 g_x, so
// the sweeps move axes and the g follow once at the end.
#include "gc_common.h"
#include "gc_internal.h"

#pragma clang fp contract(off)

namespace {

using namespace gc;

struct Quat {
    double w, x, y, z;   // q0, q1, q2, q3
};

// (i s_a)(i s_b) = -delta_ab - i eps_abc s_c
__device__ __forceinline__ Quat qmul(const Quat &p, const Quat &q)
{
    Quat r;
    r.w = p.w * q.w - p.x * q.x - p.y * q.y - p.z * q.z;
    r.x = p.w * q.x + q.w * p.x - (p.y * q.z - p.z * q.y);
    r.y = p.w * q.y + q.w * p.y - (p.z * q.x - p.x * q.z);
    r.z = p.w * q.z + q.w * p.z - (p.x * q.y - p.y * q.x);
    return r;
}

__device__ __forceinline__ Quat qconj(const Quat &q) { return Quat{q.w, -q.x, -q.y, -q.z}; }

// b with Q s3 Q^dagger = b . s: b3 = |alpha|^2 - |beta|^2, b1 - i b2 =
// -2 alpha beta for Q = [[alpha, beta], [-conj(beta), conj(alpha)]],
// alpha = q0 + i q3, beta = q2 + i q1
__device__ __forceinline__ void rot3(const Quat &q, double &b1, double &b2, double &b3)
{
    b1 = -2.0 * (q.w * q.y - q.x * q.z);
    b2 = 2.0 * (q.w * q.x + q.y * q.z);
    b3 = q.w * q.w + q.z * q.z - q.x * q.x - q.y * q.y;
}

// The g with g^dagger s3 g = n . s whose conjugate h = g^dagger has a real,
// non-negative diagonal element: alpha = sqrt((1 + n3)/2), beta =
// -(n1 - i n2)/(2 alpha) (alpha = 0, beta = 1 at n3 = -1)
__device__ __forceinline__ Quat from_axis3(double n1, double n2, double n3)
{
    const double a = sqrt(0.5 * (1.0 + n3));
    double br = 1.0, bi = 0.0;
    if (a > 0.0) {
        const double den = 2.0 * a;
        br = -n1 / den;
        bi = n2 / den;
    }
    return Quat{a, -bi, -br, -0.0};
}

__device__ __forceinline__ Quat load_q(const double *__restrict__ p, size_t k)
{
    const double4 v = reinterpret_cast<const double4 *>(p)[k];
    return Quat{v.x, v.y, v.z, v.w};
}

// (q0 + i q.s) (v.s) (q0 - i q.s) = v'.s
struct Axis {
    double x, y, z;
};
__device__ __forceinline__ Axis turn(const Quat &q, const Axis &v)
{
    const double t = 2.0 * fma(q.x, v.x, fma(q.y, v.y, q.z * v.z));
    const double s = fma(q.w, q.w, -fma(q.x, q.x, fma(q.y, q.y, q.z * q.z)));
    const double w = 2.0 * q.w;
    return Axis{fma(s, v.x, fma(t, q.x, w * fma(v.y, q.z, -(v.z * q.y)))),
                fma(s, v.y, fma(t, q.y, w * fma(v.z, q.x, -(v.x * q.z)))),
                fma(s, v.z, fma(t, q.z, w * fma(v.x, q.y, -(v.y * q.x))))};
}

constexpr int kMagBlock = 1024;     // threads with the links in global memory,
constexpr int kMagBlockReg = 768;   // at most, with the links in registers

// Sum over the workgroup in a fixed order (wavefront sums, then the waves in
// order); every thread returns the total.  One barrier; the next call's
// values reach red after another one.
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
    return t;
}

// One workgroup per configuration, the axes in LDS.  links [d][V]
// quaternions, nbr [2d][V] (forward, then backward), csite [V]: the sites of
// colour 0, then those of colour 1 (V/2 each).  A sweep updates colour 0, then
// colour 1: R depends on n_x through n . M with M = sum_mu [w_mu + y_mu] (mu
// ascending, forward then backward), w_mu the axis of x + mu turned by
// U_{x,mu} and y_mu that of x - mu turned by U_{x-mu,mu}^dagger, so n = M/|M|
// (M = 0 leaves it unchanged).  D = (1/V) sum_x |n_x - n_x^old|^2 over a
// sweep; the reduction stops after the first sweep with D < eps, or after
// max_sweeps.  Then phi[mu][x] = arg of the diagonal element of U'_{x,mu} and
// out the sweeps, R/(dV) and whether D fell below eps.
//
// One CU, so a sweep's chain counts: with REG (one site of each colour per
// thread, V <= 1536) the thread's 4d links stay in registers, 128 of 168 in
// four dimensions, and axes are stored by colour, without bank conflicts;
// larger lattices read 32 bytes per link and site update from the L2, 64
// bytes per clock.  A turned axis takes 24 double-precision instructions, the
// product of quaternions and its axis 45.  1214 sweeps of a random
// 6^4 take 6.2 ms (11.1 with quaternions and links from the L2; 3600 cycles of
// double-precision issue per colour are 3.9 of them), 1320 of 8^3 2.3 (5.6),
// 740 of 16^2 1.0 (2.3), 2189 of 8^4 43 (49).
template <int D, bool REG>
__global__ __launch_bounds__(REG ? kMagBlockReg : kMagBlock, REG ? 3 : 4) void mag_kernel(
    const double *__restrict__ links, const int *__restrict__ nbr, const int *__restrict__ csite, int V, double eps,
    uint64_t max_sweeps, double *__restrict__ phi, GcMagOut *__restrict__ out)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kMagBlock / 64];
    const int tid = (int)threadIdx.x, block = (int)blockDim.x;
    const int half = V / 2;
    // x and y of the axis at a site's place, z of all sites, then (REG) the
    // places: rank in csite
    lds_ptr<dbl2> axy = as_lds(reinterpret_cast<dbl2 *>(smem));
    lds_ptr<double> az = as_lds(reinterpret_cast<double *>(smem + 16 * (size_t)V));
    lds_ptr<uint16_t> place = as_lds(reinterpret_cast<uint16_t *>(smem + 24 * (size_t)V));
    for (int x = tid; x < V; x += block) {
        axy[x] = dbl2{0.0, 0.0};
        az[x] = 1.0;
        if (REG) place[csite[x]] = (uint16_t)x;
    }
    __syncthreads();
    auto at = [&](int x) __attribute__((always_inline)) { return REG ? (int)place[x] : x; };
    auto axis = [&](int p) __attribute__((always_inline)) {
        const dbl2 v = axy[p];
        return Axis{v.x, v.y, az[p]};
    };
    Quat u[REG ? 2 : 1][2 * D];
    uint32_t np[REG ? 2 : 1][D];   // places, forward | backward << 16
    if constexpr (REG) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int x = csite[c * half + min(tid, half - 1)];
#pragma unroll
            for (int mu = 0; mu < D; ++mu) {
                const int f = nbr[mu * V + x], b = nbr[(D + mu) * V + x];
                u[c][2 * mu] = load_q(links, (size_t)mu * V + x);
                u[c][2 * mu + 1] = qconj(load_q(links, (size_t)mu * V + b));
                np[c][mu] = (uint32_t)place[f] | ((uint32_t)place[b] << 16);
            }
        }
    }
    uint64_t sweeps = 0;
    int converged = 0;
    double acc = 0.0;
    // the new axis at place p from M
    auto update = [&](int p, const Axis &m) __attribute__((always_inline)) {
        const double mm = fma(m.x, m.x, fma(m.y, m.y, m.z * m.z));
        if (mm > 0.0) {
            const Axis o = axis(p);
            const double s = sqrt(mm);
            const Axis n = {m.x / s, m.y / s, m.z / s};
            axy[p] = dbl2{n.x, n.y};
            az[p] = n.z;
            const double e1 = n.x - o.x, e2 = n.y - o.y, e3 = n.z - o.z;
            acc += fma(e1, e1, fma(e2, e2, e3 * e3));
        }
    };
    while (sweeps < max_sweeps) {
        acc = 0.0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if constexpr (REG) {
                if (tid < half) {
                    Axis m = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int mu = 0; mu < D; ++mu) {
                        // not hoisted: a turn's link-only factors would take
                        // more registers than there are
                        Quat &uf = u[c][2 * mu], &ub = u[c][2 * mu + 1];
                        asm volatile("" : "+v"(uf.w), "+v"(uf.x), "+v"(uf.y), "+v"(uf.z));
                        asm volatile("" : "+v"(ub.w), "+v"(ub.x), "+v"(ub.y), "+v"(ub.z));
                        const uint32_t p = np[c][mu];
                        const Axis nf = axis((int)(p & 0xffff)), nb = axis((int)(p >> 16));
                        const Axis v = turn(uf, nf);
                        const Axis y = turn(ub, nb);
                        m.x = (m.x + v.x) + y.x;
                        m.y = (m.y + v.y) + y.y;
                        m.z = (m.z + v.z) + y.z;
                        if (D == 4) __builtin_amdgcn_sched_barrier(0);   // bounds the values in flight
                    }
                    update(c * half + tid, m);
                }
            } else {
                for (int j = tid; j < half; j += block) {
                    const int x = csite[c * half + j];
                    Axis m = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int mu = 0; mu < D; ++mu) {
                        const int f = nbr[mu * V + x], b = nbr[(D + mu) * V + x];
                        const Axis v = turn(load_q(links, (size_t)mu * V + x), axis(f));
                        const Axis y = turn(qconj(load_q(links, (size_t)mu * V + b)), axis(b));
                        m.x = (m.x + v.x) + y.x;
                        m.y = (m.y + v.y) + y.y;
                        m.z = (m.z + v.z) + y.z;
                    }
                    update(x, m);
                }
            }
            if (c == 0) __syncthreads();
        }
        ++sweeps;
        const double Dn = block_sum(acc, red) / (double)V;   // with the sweep's second barrier
        if (Dn < eps) {
            converged = 1;
            break;
        }
    }
    auto g = [&](int x) __attribute__((always_inline)) {
        const Axis n = axis(at(x));
        return from_axis3(n.x, n.y, n.z);
    };
    double racc = 0.0;
    for (int l = tid; l < D * V; l += block) {
        const int mu = l / V, x = l - mu * V;
        const Quat Up = qmul(qmul(g(x), load_q(links, (size_t)l)), qconj(g(nbr[mu * V + x])));
        double b1, b2, b3;
        rot3(Up, b1, b2, b3);
        racc += b3;
        phi[l] = atan2(Up.z, Up.w);
    }
    __syncthreads();   // the last sweep's sums are read
    const double R = block_sum(racc, red) / (double)(D * V);
    if (tid == 0) {
        out->sweeps = sweeps;
        out->R = R;
        out->converged = converged;
    }
}

template <int D>
void launch_mag(const double *links, const int *nbr, const int *csite, int V, double eps, uint64_t max_sweeps,
                double *phi, GcMagOut *out, hipStream_t s)
{
    const size_t lds = gc_mag_lds_bytes(V);
    if (V / 2 <= kMagBlockReg)
        hipLaunchKernelGGL((mag_kernel<D, true>), dim3(1), dim3((V / 2 + 63) / 64 * 64), lds, s, links, nbr, csite, V,
                           eps, max_sweeps, phi, out);
    else
        hipLaunchKernelGGL((mag_kernel<D, false>), dim3(1), dim3(kMagBlock), lds, s, links, nbr, csite, V, eps,
                           max_sweeps, phi, out);
}

}  // namespace

size_t gc_mag_lds_bytes(int V) { return 32 * (size_t)V; }

hipError_t gc_launch_mag(const double *links, const int *nbr, const int *csite, int d, int V, double eps,
                         uint64_t max_sweeps, double *phi, GcMagOut *out, hipStream_t s)
{
    switch (d) {
    case 1: launch_mag<1>(links, nbr, csite, V, eps, max_sweeps, phi, out, s); break;
    case 2: launch_mag<2>(links, nbr, csite, V, eps, max_sweeps, phi, out, s); break;
    case 3: launch_mag<3>(links, nbr, csite, V, eps, max_sweeps, phi, out, s); break;
    case 4: launch_mag<4>(links, nbr, csite, V, eps, max_sweeps, phi, out, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
