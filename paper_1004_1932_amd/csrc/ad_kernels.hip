/*
 * HIP kernels for gfx950 (CDNA4): the all-pairs Oseen mobility step of
 * active spring dumbbell suspensions (Putz, Dunkel, Yeomans, Sec. II and
 * Sec. V).
 *
 * In the two-kernel form one RK4 stage is two launches (the fused stage
 * kernels, the resident ones and k_pairs_f64w do both parts in one):
 *   k_pairs_*   the O(N^2) pair sum over a work list of (i-block, j-chunk)
 *               items; each item stages its j-tiles through LDS and every
 *               lane holds IPL consecutive target spheres in registers.
 *   k_epilogue  sums the j-chunk partials in chunk order, forms the stage
 *               velocity k = u0 + kappa*acc, updates the RK accumulator and
 *               the state, and evaluates the spring forces of the next stage
 *               (Eq. e:swimmer_potential) into the pack the next pair sum
 *               reads.
 * Packs are double-buffered: stage s reads one and writes the other.
 *
 * All FP64 arithmetic is written in a fixed order and built without FMA
 * contraction; FP32 FMAs are spelled out with __builtin_fmaf.
 */
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "ad_internal.h"

namespace ad {

/* ------------------------------------------------------------ helpers */

__device__ __forceinline__ void spring_forces(const Coef& c, const double y0[3], const double y1[3],
                                              double sphi, double cphi, double st, double ct,
                                              double f0[3], double f1[3]) {
    /* F_{2s+1} = -k (d - L) n/d, F_{2s} = -F_{2s+1}, n = y1 - y0,
     * L = ell + lam sin(omega t + phi) by the addition theorem. */
    double nx = y1[0] - y0[0], ny = y1[1] - y0[1], nz = y1[2] - y0[2];
    double d = sqrt((nx * nx + ny * ny) + nz * nz);
    double L = c.ell + c.lam * (st * cphi + ct * sphi);
    double cc = (-c.k * (d - L)) / d;
    f1[0] = cc * nx;
    f1[1] = cc * ny;
    f1[2] = cc * nz;
    f0[0] = -f1[0];
    f0[1] = -f1[1];
    f0[2] = -f1[2];
}

/* Oseen term of one source sphere in FP64, without the 1/(8 pi eta) factor:
 * [F/r + r (r.F)/r^3]. */
__device__ __forceinline__ void oseen_term64(const double r[3], const double F[3], double out[3]) {
    double r2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
    double ir = 1.0 / sqrt(r2);
    double fr = (r[0] * F[0] + r[1] * F[1]) + r[2] * F[2];
    double t = fr / r2;
    out[0] = ir * (F[0] + t * r[0]);
    out[1] = ir * (F[1] + t * r[1]);
    out[2] = ir * (F[2] + t * r[2]);
}

/* Rotne-Prager-Yamakawa-Mazur correction of one source sphere in FP64,
 * without its 2a^2/(24 pi eta) factor: (F - 3 r (r.F)/r^2)/r^3, in the
 * operation order of the plain sum. */
__device__ __forceinline__ void rpy_term64(const double r[3], const double F[3], double out[3]) {
    double r2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
    double ir = 1.0 / sqrt(r2);
    double fr = (r[0] * F[0] + r[1] * F[1]) + r[2] * F[2];
    double t = fr / r2;
    double ir3 = ir / r2;
    double t3 = 3.0 * t;
    out[0] = ir3 * (F[0] - t3 * r[0]);
    out[1] = ir3 * (F[1] - t3 * r[1]);
    out[2] = ir3 * (F[2] - t3 * r[2]);
}

/* Steric sum for sphere i over the spheres [j0, j1) of its system: for
 * 0 < r < rc, ks (rc - r) (X_i - X_j)/r, ascending j. Positions are read
 * through `get`. Returns non-zero if a coincident sphere was met. */
template <class Get>
__device__ int steric_sum(const Coef& c, int i, int j0, int j1, Get get, double acc[3], int* any) {
    double xi[3];
    get(i, xi);
    double rc2 = c.rc * c.rc;
    int bad = 0;
    acc[0] = acc[1] = acc[2] = 0.0;
    *any = 0;
    for (int j = j0; j < j1; ++j) {
        if (j == i) continue;
        double xj[3];
        get(j, xj);
        double rx = xi[0] - xj[0], ry = xi[1] - xj[1], rz = xi[2] - xj[2];
        double r2 = (rx * rx + ry * ry) + rz * rz;
        if (r2 >= rc2) continue;
        if (r2 == 0.0) {
            bad = 1;
            continue;
        }
        double r = sqrt(r2);
        double cc = c.ks * (c.rc - r) / r;
        acc[0] = acc[0] + cc * rx;
        acc[1] = acc[1] + cc * ry;
        acc[2] = acc[2] + cc * rz;
        *any = 1;
    }
    return bad;
}

/* The full steric sums of a dumbbell's two spheres, by one thread (IT = 0,
 * steric_sum) or by a wave for its IT spheres, IT / 2 dumbbells of one system
 * from s0 on: the lanes test 64 sources at a time, each against every sphere,
 * on the high words of r^2 and rc^2 (an FP64 compare costs as much as the
 * separation), and where one may be in reach the wave adds up the terms of the
 * lanes that pass in order, so every sum is steric_sum's, bit for bit. What
 * bounds it is the FP64 rate: 8 operations per sphere and 64 sources. Where
 * many pass (a contact distance of many radii) the terms go through LDS, added
 * by rows: one contact after another, each with its own square root and
 * division, 512 systems of 200 spheres all in reach took 2.1 ms, a thread per
 * dumbbell 0.13, so 0.11. The lanes 2m end with the forces of dumbbell
 * s0 + m. */
template <int IT>
__device__ __forceinline__ int steric_dumbbell(const Dev& d, int& s0) {
    if (IT == 0) {
        s0 = blockIdx.x * blockDim.x + threadIdx.x;
        return s0 < d.Stot ? s0 : -1;
    }
    const int lane = threadIdx.x & 63;
    s0 = __builtin_amdgcn_readfirstlane((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (IT / 2));
    return (lane & 1) == 0 && lane < IT && s0 + (lane >> 1) < d.Stot ? s0 + (lane >> 1) : -1;
}
__device__ __forceinline__ double read_lane(double v, int l) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, l), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), l);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
/* adds the steric forces of dumbbell s (from steric_dumbbell) to f0 and f1 */
template <int IT, class Get>
__device__ __forceinline__ int add_steric(const Dev& d, const Coef& c, int s, int s0, Get get, double f0[3],
                                          double f1[3]) {
    int bad = 0;
    if (IT == 0) {
        const int b = d.dsys[s], j0 = d.sys_off[b], j1 = d.sys_off[b + 1];
        double acc[3];
        int any;
        bad |= steric_sum(c, 2 * s, j0, j1, get, acc, &any);
        if (any)
            for (int a = 0; a < 3; ++a) f0[a] = f0[a] + acc[a];
        bad |= steric_sum(c, 2 * s + 1, j0, j1, get, acc, &any);
        if (any)
            for (int a = 0; a < 3; ++a) f1[a] = f1[a] + acc[a];
        return bad;
    }
    if (s0 >= d.Stot) return 0;
    constexpr int NQ = IT ? IT : 1;
    const int lane = threadIdx.x & 63;
    const int b = d.dsys[s0], j0 = d.sys_off[b], j1 = d.sys_off[b + 1];
    const int nq = min(NQ, 2 * (d.Stot - s0));
    const double rc2 = c.rc * c.rc;
    const unsigned reach = (unsigned)(__builtin_bit_cast(unsigned long long, rc2) >> 32);
    double xi[NQ][3];
#pragma unroll
    for (int q = 0; q < NQ; ++q) get(2 * s0 + min(q, nq - 1), xi[q]);
    /* lane 3 q + a adds up component a of sphere q */
    const int mine = lane / 3, a_r = lane - 3 * mine;
    __shared__ __align__(16) double rows[4][6][66]; /* per wave; rows of pairs of columns */
    double(*row)[66] = rows[threadIdx.x >> 6];
    double acc = 0.0;
    bool any = false;
    double xj[3], xn[3];
    get(min(j0 + lane, j1 - 1), xn);
    for (int jt = j0; jt < j1; jt += 64) {
        for (int a = 0; a < 3; ++a) xj[a] = xn[a];
        if (jt + 64 < j1) get(min(jt + 64 + lane, j1 - 1), xn);
        unsigned lo = 0xffffffffu, hi = 0; /* of the high words; NaN's are above infinity's */
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double rx = xi[q][0] - xj[0], ry = xi[q][1] - xj[1], rz = xi[q][2] - xj[2];
            const double r2 = (rx * rx + ry * ry) + rz * rz;
            const unsigned h = (unsigned)(__builtin_bit_cast(unsigned long long, r2) >> 32) & 0x7fffffffu;
            lo = min(lo, h);
            hi = max(hi, h);
        }
        if (!__any(lo <= reach || hi >= 0x7ff00000u)) continue;
        const int j = jt + lane;
#pragma unroll 1
        for (int q = 0; q < nq; q += 2) { /* a dumbbell's two spheres */
            double t[2][3], t2[2];
            unsigned long long in[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                double y[3];
                get(2 * s0 + q + u, y);
                for (int a = 0; a < 3; ++a) t[u][a] = y[a] - xj[a];
                t2[u] = (t[u][0] * t[u][0] + t[u][1] * t[u][1]) + t[u][2] * t[u][2];
                const bool near = j < j1 && j != 2 * s0 + q + u && !(t2[u] >= rc2);
                in[u] = __ballot(near && t2[u] != 0.0);
                if (__any(near && t2[u] == 0.0)) bad = 1;
                any |= mine == q + u && in[u] != 0;
            }
            if (!(in[0] | in[1])) continue;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double r = sqrt(t2[u]);
                const double cc = c.ks * (c.rc - r) / r;
                for (int a = 0; a < 3; ++a) t[u][a] = cc * t[u][a];
            }
            if (__popcll(in[0]) + __popcll(in[1]) > 16) {
                /* many: by rows through LDS, +0.0 for the lanes that do not pass
                 * (a sum that started at +0.0 does not change by it) */
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    for (int a = 0; a < 3; ++a) row[3 * u + a][lane] = (in[u] >> lane & 1) ? t[u][a] : 0.0;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int o = lane - 3 * q;
                const double2* v = reinterpret_cast<const double2*>(row[o < 0 ? 0 : o > 5 ? 5 : o]);
                double sum = acc;
#pragma unroll 4
                for (int k = 0; k < 32; ++k) {
                    sum = sum + v[k].x;
                    sum = sum + v[k].y;
                }
                if (o >= 0 && o < 6) acc = sum;
                continue;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                unsigned long long m = in[u];
                while (m) {
                    const int l = __builtin_ctzll(m);
                    m &= m - 1;
                    const double x = read_lane(t[u][0], l), y = read_lane(t[u][1], l), z = read_lane(t[u][2], l);
                    const double sum = acc + (a_r == 0 ? x : a_r == 1 ? y : z);
                    acc = mine == q + u ? sum : acc;
                }
            }
        }
    }
    /* to the lanes 2 m, which hold dumbbell s0 + m */
    const int from = 3 * lane;
    const bool any0 = __shfl((int)any, from & 63), any1 = __shfl((int)any, (from + 3) & 63);
    for (int a = 0; a < 3; ++a) {
        const double g0 = __shfl(acc, (from + a) & 63), g1 = __shfl(acc, (from + 3 + a) & 63);
        if (any0) f0[a] = f0[a] + g0;
        if (any1) f1[a] = f1[a] + g1;
    }
    return bad;
}

__device__ __forceinline__ void split_f32(double v, float& hi, float& lo) {
    hi = (float)v;
    lo = (float)(v - (double)hi);
}

/* (hi, lo) += v with TwoSum: hi + lo keeps the exact sum up to the rounding
 * of lo. */
__device__ __forceinline__ void two_sum_acc(float& hi, float& lo, float v) {
    const float s = hi + v;
    const float bb = s - hi;
    const float e = (hi - (s - bb)) + (v - bb);
    hi = s;
    lo = lo + e;
}


/* 1/sqrt(r2) from v_rsq_f64 (about 2^-24) and one third-order step
 * y (1 + e/2 + 3 e^2/8), e = 1 - r2 y^2: within an ulp. (One Newton step, two
 * instructions fewer, leaves 4e-15.) */
__device__ __forceinline__ double rsqrt64(double r2) {
    const double y = __builtin_amdgcn_rsq(r2);
    const double g = r2 * y;
    const double e = __builtin_fma(-g, y, 1.0);
    const double p = __builtin_fma(e, 0.375, 0.5);
    return __builtin_fma(y * e, p, y);
}

/* Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
 * 32x32->64 multiplications by the published multipliers, the key bumped by
 * the Weyl constants between rounds. */
__device__ __forceinline__ void philox4x32_10(unsigned c[4], unsigned k0, unsigned k1) {
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const unsigned hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
        const unsigned hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
        const unsigned n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
}

/* log u for u in (0, 1), within two ulp: u = 2^e m, m in [sqrt(1/2), sqrt(2)),
 * log m = 2 atanh(q), q = (m - 1)/(m + 1), by the series of atanh up to q^23
 * (|q| < 0.172: the next term is below 2^-63). */
__device__ __forceinline__ double log_unit(double u) {
    double m = __builtin_amdgcn_frexp_mant(u); /* in [1/2, 1) */
    int e = __builtin_amdgcn_frexp_exp(u);
    const bool low = m < 0.70710678118654757;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0, g = m + 1.0;
    double y = __builtin_amdgcn_rcp(g);
    y = __builtin_fma(y, __builtin_fma(-g, y, 1.0), y);
    double q = f * y;
    q = __builtin_fma(__builtin_fma(-g, q, f), y, q);
    const double z = q * q;
    double p = 1.0 / 23.0;
    p = __builtin_fma(p, z, 1.0 / 21.0);
    p = __builtin_fma(p, z, 1.0 / 19.0);
    p = __builtin_fma(p, z, 1.0 / 17.0);
    p = __builtin_fma(p, z, 1.0 / 15.0);
    p = __builtin_fma(p, z, 1.0 / 13.0);
    p = __builtin_fma(p, z, 1.0 / 11.0);
    p = __builtin_fma(p, z, 1.0 / 9.0);
    p = __builtin_fma(p, z, 1.0 / 7.0);
    p = __builtin_fma(p, z, 1.0 / 5.0);
    p = __builtin_fma(p, z, 1.0 / 3.0);
    const double q2 = q + q;
    /* e log 2 in two parts: the first product is exact (log 2 to 36 bits) */
    const double lo = __builtin_fma((double)e, 0x1.cf79abc9e3b3ap-40, (q2 * z) * p);
    return __builtin_fma((double)e, 0x1.62e42fefa0000p-1, q2 + lo);
}

/* sin (a = 1) or cos of 2 pi u, u in (0, 1) a multiple of 2^-33: the turn is
 * reduced exactly by quarters to |t| <= 1/8, then Taylor polynomials of
 * 2 pi t (the next terms are below 2^-57). */
__device__ __forceinline__ double trig_turn(double u, int a) {
    const double k = __builtin_rint(4.0 * u);
    const double x = (u - 0.25 * k) * 6.283185307179586477;
    const double z = x * x;
    double s = 1.0 / 355687428096000.0;
    s = __builtin_fma(s, z, -1.0 / 1307674368000.0);
    s = __builtin_fma(s, z, 1.0 / 6227020800.0);
    s = __builtin_fma(s, z, -1.0 / 39916800.0);
    s = __builtin_fma(s, z, 1.0 / 362880.0);
    s = __builtin_fma(s, z, -1.0 / 5040.0);
    s = __builtin_fma(s, z, 1.0 / 120.0);
    s = __builtin_fma(s, z, -1.0 / 6.0);
    s = __builtin_fma(x * z, s, x);
    double c = 1.0 / 20922789888000.0;
    c = __builtin_fma(c, z, -1.0 / 87178291200.0);
    c = __builtin_fma(c, z, 1.0 / 479001600.0);
    c = __builtin_fma(c, z, -1.0 / 3628800.0);
    c = __builtin_fma(c, z, 1.0 / 40320.0);
    c = __builtin_fma(c, z, -1.0 / 720.0);
    c = __builtin_fma(c, z, 1.0 / 24.0);
    c = __builtin_fma(c, z, -0.5);
    c = __builtin_fma(c, z, 1.0);
    /* cos is sin a quarter turn on */
    const int n = (int)k + (a == 1 ? 0 : 1);
    const double v = (n & 1) ? c : s;
    const unsigned long long sign = (unsigned long long)((n >> 1) & 1) << 63;
    return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, v) ^ sign);
}

/* Standard normal component a (0..2) of sphere i at step n: Box-Muller on
 * the four uniforms (x + 1/2) 2^-32 of one Philox block with counter
 * (i, n) and key seed. (With the library's log, sin and cos, made for any
 * operand, the 1354-sphere Heun step with noise took 3.5 us more.) */
__device__ __forceinline__ double gauss_component(unsigned long long seed, int i, long long n, int a) {
    unsigned c[4] = {(unsigned)i, (unsigned)n, (unsigned)((unsigned long long)n >> 32), 0u};
    philox4x32_10(c, (unsigned)seed, (unsigned)(seed >> 32));
    const double u0 = ((double)(a == 2 ? c[2] : c[0]) + 0.5) * 0x1p-32;
    const double u1 = ((double)(a == 2 ? c[3] : c[1]) + 0.5) * 0x1p-32;
    const double x = -2.0 * log_unit(u0); /* in [2^-32, 46] */
    double y = rsqrt64(x), r = x * y;
    r = __builtin_fma(__builtin_fma(-r, r, x), 0.5 * y, r);
    return r * trig_turn(u1, a);
}

/* The noise of component a of sphere i in both stages of Heun step n. */
__device__ __forceinline__ double stage_noise(const Coef& c, int i, long long n, int a) {
    return c.noise ? c.g * gauss_component(c.seed, i, n, a) : 0.0;
}

/* Write the pair-kernel pack and the self (+partner) velocity u0 of the two
 * spheres of one dumbbell at positions y0, y1 with forces f0, f1; into the
 * next-stage pack buffers when nxt != 0. */
/* FP32C pack of sphere i at stage position y with spring force f, its
 * dumbbell partner at yp with force fp: u0 = self term plus the partner's
 * term in FP64 (the pair kernels skip the partner), then the FP32 hi/lo
 * position and force: A = (hi.xyz, Fx), B = (lo.xyz, Fy), C = (Fy, Fz), so
 * that a reader of single-float positions needs A and C only. */
__device__ __forceinline__ void store_pack_sphere(const Dev& d, const Coef& c, int i, const double y[3],
                                                  const double yp[3], const double f[3], const double fp[3],
                                                  int nxt) {
    const int N = d.Ntot;
    const double r[3] = {y[0] - yp[0], y[1] - yp[1], y[2] - yp[2]};
    double t[3], q[3];
    oseen_term64(r, fp, t);
    if (c.rpy) rpy_term64(r, fp, q);
    for (int a = 0; a < 3; ++a) {
        double u = c.cs * f[a] + c.co * t[a];
        if (c.rpy) u = u + c.cr * q[a];
        d.U0[a * N + i] = u;
    }
    float h[3], l[3];
    for (int a = 0; a < 3; ++a) split_f32(y[a], h[a], l[a]);
    (nxt ? d.pA2 : d.pA)[i] = make_float4(h[0], h[1], h[2], (float)f[0]);
    (nxt ? d.pB2 : d.pB)[i] = make_float4(l[0], l[1], l[2], (float)f[1]);
    (nxt ? d.pC2 : d.pC)[i] = make_float2((float)f[1], (float)f[2]);
}

/* The closing update of the FP32C stage kernels uses these two forms of
 * spring_forces and store_pack_sphere: one rsqrt64 (within an ulp) in place
 * of the IEEE square roots and divisions; r = y - yp is +-(y1 - y0) exactly,
 * so the partner term takes the spring's 1/d. In the FP32C path the state stays FP64 and
 * only the pair sums are FP32, so a relative error near 1e-16 here is far
 * below theirs (about 1e-7); the FP64 paths keep the IEEE forms, whose
 * operation order the bitwise parity with the plain sum depends on. With
 * single-float positions (SPLIT = 0) no stage kernel reads the lo parts, so
 * B is not written. spring_forces_rs returns the 1/d it used. */
__device__ __forceinline__ double spring_forces_rs(const Coef& c, const double y0[3], const double y1[3],
                                                   double sphi, double cphi, double st, double ct,
                                                   double f0[3], double f1[3]) {
    /* -k (d - L) n / d = k (L / d - 1) n */
    const double nx = y1[0] - y0[0], ny = y1[1] - y0[1], nz = y1[2] - y0[2];
    const double id = rsqrt64((nx * nx + ny * ny) + nz * nz);
    const double L = c.ell + c.lam * (st * cphi + ct * sphi);
    const double cc = c.k * (L * id - 1.0);
    f1[0] = cc * nx;
    f1[1] = cc * ny;
    f1[2] = cc * nz;
    f0[0] = -f1[0];
    f0[1] = -f1[1];
    f0[2] = -f1[2];
    return id;
}

template <int SPLIT>
__device__ __forceinline__ void store_pack_sphere_rs(const Dev& d, const Coef& c, int i, const double y[3],
                                                     const double yp[3], const double f[3], const double fp[3],
                                                     double ir) {
    const int N = d.Ntot;
    const double r[3] = {y[0] - yp[0], y[1] - yp[1], y[2] - yp[2]};
    const double ir2 = ir * ir;
    const double t = ((r[0] * fp[0] + r[1] * fp[1]) + r[2] * fp[2]) * ir2;
    for (int a = 0; a < 3; ++a) {
        double u = c.cs * f[a] + c.co * (ir * (fp[a] + t * r[a]));
        if (c.rpy) u = u + c.cr * ((ir * ir2) * (fp[a] - (3.0 * t) * r[a]));
        d.U0[a * N + i] = u;
    }
    float h[3], l[3];
    for (int a = 0; a < 3; ++a) split_f32(y[a], h[a], l[a]);
    d.pA2[i] = make_float4(h[0], h[1], h[2], (float)f[0]);
    if (SPLIT) d.pB2[i] = make_float4(l[0], l[1], l[2], (float)f[1]);
    d.pC2[i] = make_float2((float)f[1], (float)f[2]);
}

__device__ void store_pack(const Dev& d, const Coef& c, int prec, int i0, const double y0[3],
                           const double y1[3], const double f0[3], const double f1[3], int nxt) {
    const int N = d.Ntot;
    const int i1 = i0 + 1;
    if (prec == PREC_FP32C) {
        store_pack_sphere(d, c, i0, y0, y1, f0, f1, nxt);
        store_pack_sphere(d, c, i1, y1, y0, f1, f0, nxt);
    } else {
        for (int a = 0; a < 3; ++a) {
            d.U0[a * N + i0] = c.cs * f0[a];
            d.U0[a * N + i1] = c.cs * f1[a];
        }
        double2* pD = nxt ? d.pD2 : d.pD;
        pD[3 * i0 + 0] = make_double2(y0[0], y0[1]);
        pD[3 * i0 + 1] = make_double2(y0[2], f0[0]);
        pD[3 * i0 + 2] = make_double2(f0[1], f0[2]);
        pD[3 * i1 + 0] = make_double2(y1[0], y1[1]);
        pD[3 * i1 + 1] = make_double2(y1[2], f1[0]);
        pD[3 * i1 + 2] = make_double2(f1[1], f1[2]);
    }
}

/* ------------------------------------------------------------ small kernels */

__global__ void k_set_step(Ctl* ctl, long long v) { ctl->slot[0] = v; }
__global__ void k_clear_flag(Ctl* ctl) { ctl->flag = 0; }

__global__ void k_state_in(Dev d, const double* __restrict__ Xa) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d.Ntot) return;
    for (int a = 0; a < 3; ++a) d.X[a * d.Ntot + i] = Xa[3 * i + a];
}

__global__ void k_state_out(Dev d, double* __restrict__ Xa) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d.Ntot) return;
    for (int a = 0; a < 3; ++a) Xa[3 * i + a] = d.X[a * d.Ntot + i];
}

/* empty every steric candidate list */
__global__ void k_clear_counts(Dev d) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d.Ntot || !d.nbr_cnt) return;
    d.nbr_cnt[i] = 0;
}

/* pack from the state at time (st, ct); spring (+ steric) forces */
template <int IT>
__global__ __launch_bounds__(256) void k_pack_state(Dev d, Coef c, int prec, double st, double ct) {
    int s0;
    const int s = steric_dumbbell<IT>(d, s0);
    if (IT == 0 && s < 0) return;
    const int N = d.Ntot;
    const int i0 = 2 * max(s, 0);
    double y0[3], y1[3], f0[3], f1[3];
    for (int a = 0; a < 3; ++a) {
        y0[a] = d.X[a * N + i0];
        y1[a] = d.X[a * N + i0 + 1];
    }
    double2 tp = d.phitrig[max(s, 0)];
    spring_forces(c, y0, y1, tp.x, tp.y, st, ct, f0, f1);
    if (c.ks != 0.0) {
        auto get = [&](int j, double x[3]) {
            x[0] = d.X[j];
            x[1] = d.X[N + j];
            x[2] = d.X[2 * N + j];
        };
        if (add_steric<IT>(d, c, s, s0, get, f0, f1)) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
        if (s < 0) return;
        /* stage positions (for the displacement check) and empty candidate
         * lists for the first pair sum */
        for (int a = 0; a < 3; ++a) {
            d.Y[a * N + i0] = y0[a];
            d.Y[a * N + i0 + 1] = y1[a];
        }
        if (d.nbr_cnt) {
            d.nbr_cnt[i0] = 0;
            d.nbr_cnt[i0 + 1] = 0;
        }
    }
    store_pack(d, c, prec, i0, y0, y1, f0, f1, 0);
}

/* pack from caller positions and forces (row-major [N][3]) */
__global__ void k_pack_apply(Dev d, Coef c, int prec, const double* __restrict__ Xa,
                             const double* __restrict__ Fa) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= d.Stot) return;
    const int i0 = 2 * s;
    double y0[3], y1[3], f0[3], f1[3];
    for (int a = 0; a < 3; ++a) {
        y0[a] = Xa[3 * i0 + a];
        y1[a] = Xa[3 * i0 + 3 + a];
        f0[a] = Fa[3 * i0 + a];
        f1[a] = Fa[3 * i0 + 3 + a];
    }
    store_pack(d, c, prec, i0, y0, y1, f0, f1, 0);
}

/* spring + steric forces at caller positions, row-major output */
template <int IT>
__global__ __launch_bounds__(256) void k_forces(Dev d, Coef c, const double* __restrict__ Xa, double st, double ct,
                                                double* __restrict__ Fa) {
    int s0;
    const int s = steric_dumbbell<IT>(d, s0);
    if (IT == 0 && s < 0) return;
    const int i0 = 2 * max(s, 0);
    double y0[3], y1[3], f0[3], f1[3];
    for (int a = 0; a < 3; ++a) {
        y0[a] = Xa[3 * i0 + a];
        y1[a] = Xa[3 * i0 + 3 + a];
    }
    double2 tp = d.phitrig[max(s, 0)];
    spring_forces(c, y0, y1, tp.x, tp.y, st, ct, f0, f1);
    if (c.ks != 0.0) {
        auto get = [&](int j, double x[3]) {
            x[0] = Xa[3 * j];
            x[1] = Xa[3 * j + 1];
            x[2] = Xa[3 * j + 2];
        };
        if (add_steric<IT>(d, c, s, s0, get, f0, f1)) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
        if (s < 0) return;
    }
    for (int a = 0; a < 3; ++a) {
        Fa[3 * i0 + a] = f0[a];
        Fa[3 * i0 + 3 + a] = f1[a];
    }
}

/* ------------------------------------------------------------ epilogue */

/* Stage update of one state component o = a N + i from its velocity k (and
 * the step's noise nz):
 * RK4 keeps the weighted sum of the stage velocities in R and writes X at the
 * last stage; Heun adds the same noise in both stages. Returns the position
 * at which the next stage evaluates the velocity. */
__device__ __forceinline__ double stage_update(const Dev& d, const Epi& e, int o, double k,
                                               double x, double r, double nz) {
    const Coef& c = e.c;
    const int stage = e.stage;
    double y;
    if (e.integ == 0) { /* RK4 */
        if (stage == 0) {
            d.R[o] = k;
            y = x + c.h2 * k;
        } else if (stage == 1) {
            d.R[o] = r + 2.0 * k;
            y = x + c.h2 * k;
        } else if (stage == 2) {
            d.R[o] = r + 2.0 * k;
            y = x + c.dt * k;
        } else {
            y = x + c.dt6 * (r + k);
            d.X[o] = y;
        }
    } else { /* Heun, with the same noise in both stages */
        if (stage == 0) {
            d.R[o] = k;
            y = x + c.dt * k;
        } else {
            y = x + c.h2 * (r + k);
        }
        if (c.noise) y = y + nz;
        if (stage == 1) d.X[o] = y;
    }
    return y;
}

constexpr int EPI_MAXP = 16; /* partials loaded per batch */

/* p[0] + p[stride] + ... of P partial sums, in order: the loads of a batch go
 * ahead of its additions (one product of 6000 spheres with RPY, whose second
 * sum was added load by load: 65.4 us, 59.6 this way; batches of 32 and 64 are
 * no faster). */
__device__ __forceinline__ double sum_slots(const double* p, long long stride, int P) {
    double v[EPI_MAXP];
#pragma unroll
    for (int q = 0; q < EPI_MAXP; ++q) v[q] = (q < P) ? p[q * stride] : 0.0;
    double acc = v[0];
#pragma unroll
    for (int q = 1; q < EPI_MAXP; ++q)
        if (q < P) acc = acc + v[q];
    for (int cc = EPI_MAXP; cc < P; cc += EPI_MAXP) {
#pragma unroll
        for (int q = 0; q < EPI_MAXP; ++q) v[q] = p[min(cc + q, P - 1) * stride];
#pragma unroll
        for (int q = 0; q < EPI_MAXP; ++q)
            if (cc + q < P) acc = acc + v[q];
    }
    return acc;
}

/* Epilogue of the spheres [i0, i0 + ni) (ni even), run by all blockDim.x
 * threads of a work-group.
 * Phase 1, one thread per sphere component: issue the loads of that
 * component's j-chunk partials, u0, X and R together, sum the partials in
 * chunk order, form k = u0 + kappa*acc and apply the (componentwise) RK
 * update: R, X to global memory, the next stage position y to LDS.
 * Phase 2, one thread per dumbbell: the next stage's spring forces at y and
 * the next pack (or, with steric forces, y and the spring forces for the
 * steric kernel). `step` numbers the noise of the Heun integrator; ys and
 * mv are LDS scratch of ni x 3 doubles. */
__device__ void epi_block(const Dev& d, const Epi& e, int i0, int ni, long long step, double (*ys)[3],
                          double (*mv)[3], int* badf) {
    const int N = d.Ntot;
    const int t = threadIdx.x;
    const int nt = blockDim.x;
    const Coef& c = e.c;
    const int stage = e.stage;
    const bool apply = (e.u_aos != nullptr);
    /* the second pass's inputs are loaded first, so their latency overlaps
     * the partial-sum loads: (sin, cos) of omega t for the next stage's
     * forces (left by this stage's pair kernel), and the phase of this
     * thread's dumbbell */
    double st = 0.0, ct = 0.0;
    double2 tp = make_double2(0.0, 0.0);
    if (!apply) {
        st = d.ctl->trig[stage][0];
        ct = d.ctl->trig[stage][1];
        if (t < ni / 2) tp = d.phitrig[(i0 >> 1) + t];
    }
    if (t == 0) *badf = 0;
    __syncthreads();
    for (int idx = t; idx < 3 * ni; idx += nt) {
        const int sl = idx / 3, a = idx - 3 * sl;
        const int i = i0 + sl;
        const int b = d.dsys[i >> 1];
        const int off = d.sys_off[b];
        const int Nb = d.sys_off[b + 1] - off;
        int P = d.sys_P[b];
        long long stride = (long long)d.ncomp * Nb;
        const double* p = d.part + d.sys_pbase[b] + (long long)a * Nb + (i - off);
        if (d.nsym && !apply) { /* the symmetric pair sum's slots of the sphere's block */
            const int bs = d.sym_bs, B = i / bs;
            P = d.sym_P[B];
            stride = 3LL * bs;
            p = d.part + d.sym_base[B] + (long long)a * bs + (i - B * bs);
        }
        const int o = a * N + i;
        /* independent loads first, so they are in flight together */
        const double u0 = d.U0[o];
        const double x = apply ? 0.0 : d.X[o];
        const double r = (!apply && stage > 0) ? d.R[o] : 0.0;
        const double yold = (!apply && !e.pack_next && d.nbr_cnt) ? d.Y[o] : 0.0;
        const double acc = sum_slots(p, stride, P);
        double k = u0 + c.co * acc;
        if (d.ncomp == 6) {
            /* FP64 with RPY: the correction's partial sums follow the Oseen
             * ones, added after them as in the plain sum */
            k = k + c.cr * sum_slots(p + 3LL * Nb, stride, P);
        }
        if (!isfinite(k)) *badf = 1;
        if (apply) {
            e.u_aos[3 * i + a] = k;
            continue;
        }
        const double y = stage_update(d, e, o, k, x, r, apply ? 0.0 : stage_noise(c, i, step, a));
        ys[sl][a] = y;
        const double dd = y - yold;
        mv[sl][a] = dd * dd;
    }
    __syncthreads();
    if (t == 0 && *badf) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (apply) return;
    /* forces of the next stage, one thread per dumbbell (ni/2 <= blockDim) */
    if (t < ni / 2) {
        const int q = t;
        const int ia = i0 + 2 * q;
        double y[2][3];
        for (int h = 0; h < 2; ++h)
            for (int a = 0; a < 3; ++a) y[h][a] = ys[2 * q + h][a];
        double f0[3], f1[3];
        spring_forces(c, y[0], y[1], tp.x, tp.y, st, ct, f0, f1);
        if (e.pack_next) {
            store_pack(d, c, e.prec, ia, y[0], y[1], f0, f1, 1);
        } else {
            if (d.nbr_cnt) {
                /* candidate lists are valid while no sphere moves more than
                 * half the skin between stage positions */
                for (int h = 0; h < 2; ++h) {
                    const double e2 = (mv[2 * q + h][0] + mv[2 * q + h][1]) + mv[2 * q + h][2];
                    if (!(e2 <= d.move2)) atomicOr(&d.ctl->flag, FLAG_NBR_SKIN);
                }
            }
            for (int a = 0; a < 3; ++a) {
                d.Y[a * N + ia] = y[0][a];
                d.Y[a * N + ia + 1] = y[1][a];
                d.Fs[a * N + ia] = f0[a];
                d.Fs[a * N + ia + 1] = f1[a];
            }
        }
    }
}

/* the epilogue as its own kernel: EPI_S spheres per work-group of EPI_T
 * threads; the step index comes from the slot the pair kernel left for this
 * stage */
constexpr int EPI_S = 32;
constexpr int EPI_T = 96;
static_assert(EPI_S / 2 <= EPI_T, "one thread per dumbbell in the second pass");

__global__ __launch_bounds__(EPI_T) void k_epilogue(Dev d, Epi e) {
    __shared__ double ys[EPI_S][3];
    __shared__ double mv[EPI_S][3];
    __shared__ int badf;
    const int i0 = blockIdx.x * EPI_S;
    const int ni = min(EPI_S, d.Ntot - i0);
    /* the step index only numbers the noise of the Heun integrator */
    const long long step = (e.u_aos || !e.c.noise) ? 0 : d.ctl->slot[e.stage & 1];
    epi_block(d, e, i0, ni, step, ys, mv, &badf);
}

/* ------------------------------------------------------------ pair sums */

/* Accumulate one FP32 pair term given ir = 1/r (0 for a skipped pair):
 * Oseen: ir (F + t r), t = (r.F) ir^2; with RPY (c' = 2a^2/3):
 * F (ir + c' ir^3) + r t (ir - 3 c' ir^3). */
template <int RPY>
__device__ __forceinline__ void pair_term(float ir, float rx, float ry, float rz, float Fx, float Fy, float Fz,
                                          float crr, float& px, float& py, float& pz) {
    const float fr = __builtin_fmaf(rz, Fz, __builtin_fmaf(ry, Fy, rx * Fx));
    const float ir2 = ir * ir;
    const float tt = fr * ir2;
    if (RPY) {
        const float ir3 = ir * ir2;
        const float av = __builtin_fmaf(crr, ir3, ir);
        const float bv = tt * __builtin_fmaf(-3.0f * crr, ir3, ir);
        px = __builtin_fmaf(av, Fx, __builtin_fmaf(bv, rx, px));
        py = __builtin_fmaf(av, Fy, __builtin_fmaf(bv, ry, py));
        pz = __builtin_fmaf(av, Fz, __builtin_fmaf(bv, rz, pz));
    } else {
        px = __builtin_fmaf(ir, __builtin_fmaf(tt, rx, Fx), px);
        py = __builtin_fmaf(ir, __builtin_fmaf(tt, ry, Fy), py);
        pz = __builtin_fmaf(ir, __builtin_fmaf(tt, rz, Fz), pz);
    }
}

/* A lane's target position in the fused stage kernels (lo: hi/lo positions only) */
struct Target {
    float hx, hy, hz, lx, ly, lz;
};

/* G = 4 (or 2) terms of a fused stage, from the LDS entries x0, x0 + dx, ...;
 * with MASK but for those of dumbbell `skip`. Their v_rsq_f32 together, see
 * rsq4. */
template <int SPLIT, int RPY, int PRIO, int MASK = 0, int G = 4>
__device__ __forceinline__ void group_terms(const Target& t, const float4* sA, const float4* sB, const float* sC,
                                           const float2* sF, int x0, int dx, float crr, float& px, float& py,
                                           float& pz, int skip = 0) {
    float rx[G], ry[G], rz[G], fx[G], fy[G], fz[G], ir[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
        const int x = x0 + u * dx;
        const float4 A = sA[x];
        fx[u] = A.w;
        if (SPLIT) {
            const float4 B = sB[x];
            fy[u] = B.w;
            fz[u] = sC[x];
            rx[u] = (t.hx - A.x) + (t.lx - B.x);
            ry[u] = (t.hy - A.y) + (t.ly - B.y);
            rz[u] = (t.hz - A.z) + (t.lz - B.z);
        } else {
            const float2 f = sF[x];
            fy[u] = f.x;
            fz[u] = f.y;
            rx[u] = t.hx - A.x;
            ry[u] = t.hy - A.y;
            rz[u] = t.hz - A.z;
        }
        ir[u] = __builtin_fmaf(rz[u], rz[u], __builtin_fmaf(ry[u], ry[u], rx[u] * rx[u]));
    }
    if (G == 4)
        rsq4<PRIO>(ir);
    else
        rsq2<PRIO>(ir);
    if (MASK) {
#pragma unroll
        for (int u = 0; u < G; ++u) ir[u] = ((x0 + u * dx) >> 1) == skip ? 0.f : ir[u];
    }
#pragma unroll
    for (int u = 0; u < G; ++u) pair_term<RPY>(ir[u], rx[u], ry[u], rz[u], fx[u], fy[u], fz[u], crr, px, py, pz);
}

/* One thread's entry of a source tile: sphere t0 + t of the pack, or
 * padding (far away and force-free, so it contributes exactly zero). */
__device__ __forceinline__ void load_tile_entry(const Dev& d, int t0, int jend, int t, float4& A, float4& B,
                                                float& C) {
    if (t0 + t < jend) {
        A = d.pA[t0 + t];
        B = d.pB[t0 + t];
        C = d.pC[t0 + t].y;
    } else {
        A = make_float4(1.0e15f, 1.0e15f, 1.0e15f, 0.f);
        B = make_float4(0.f, 0.f, 0.f, 0.f);
        C = 0.f;
    }
}

/* FP32C pair sum. A work-group of WG threads is WI x WJ waves: WI waves own
 * different target spheres (IPL consecutive spheres per lane), and the WJ
 * waves that share the same targets take interleaved parts of every j-tile.
 * A tile of WG source spheres is staged through LDS once and read as
 * broadcasts.
 *   SPLIT = 1: positions are hi + lo floats, r = (hi_i - hi_j) + (lo_i - lo_j)
 *              (r rounded relative to itself).
 *   SPLIT = 0: positions are single floats, r = x_i - x_j (error ~ eps |x|).
 * Pair math in FP32 with the hardware reciprocal square root. Each wave sums
 * the terms of one tile in FP32 and adds that tile sum to a (hi, lo)
 * accumulator with TwoSum; the WJ waves' accumulators are combined in LDS
 * in a fixed order. The dumbbell's own two spheres are skipped (their terms
 * are in u0, in FP64).
 *   STERIC = 1: every pair closer than rc + skin (r^2 is at hand) is appended
 *              to the target's candidate list for the next stage's steric
 *              forces.
 *   RPY = 1: the pair tensor carries the Rotne-Prager-Yamakawa-Mazur
 *              correction, summed with the Oseen part as
 *              F (ir + c' ir^3) + r t (ir - 3 c' ir^3), c' = 2a^2/3.
 * mode: 0 = mobility apply, 1 = step stage. */
template <int WG, int IPL, int WJ, int SPLIT, int STERIC, int RPY>
__global__ __launch_bounds__(WG) void k_pairs_f32c(Dev d, Epi e, int mode) {
    constexpr int WI = WG / 64 / WJ;
    constexpr int TJ = WG;          /* j per LDS tile */
    constexpr int IB = 64 * WI * IPL;
    /* one LDS area, used in turn by the source tiles and the cross-wave
     * combination (a barrier separates the uses) */
    union Lds {
        struct {
            float4 A[TJ];
            float4 B[TJ];
            float C[TJ];
        } tile;
        float red[WJ > 1 ? WJ : 1][IB][6];
    };
    __shared__ Lds lds;
    float4* sA = lds.tile.A;
    float4* sB = lds.tile.B;
    float* sC = lds.tile.C;
    const Item it = d.items[blockIdx.x];
    if (mode) advance_slots(d, e);
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wi = wave % WI;
    const int wj = wave / WI;
    const int slot = wi * 64 + lane;          /* target slot inside the block */
    const int ib = it.i0 + slot * IPL;
    const int iend = it.i0 + it.ni;

    float hx[IPL], hy[IPL], hz[IPL], lx[IPL], ly[IPL], lz[IPL];
    float ax[IPL], ay[IPL], az[IPL];  /* running (hi) sums */
    float bx[IPL], by[IPL], bz[IPL];  /* compensation (lo) */
    float px[IPL], py[IPL], pz[IPL];  /* tile partial */
    int dq[IPL];                      /* dumbbell of each target */
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        const int i = ib + q;
        float4 A = make_float4(0.f, 0.f, 0.f, 0.f), B = A;
        if (i < iend) {
            A = d.pA[i];
            B = d.pB[i];
        }
        hx[q] = A.x; hy[q] = A.y; hz[q] = A.z;
        lx[q] = SPLIT ? B.x : 0.f; ly[q] = SPLIT ? B.y : 0.f; lz[q] = SPLIT ? B.z : 0.f;
        ax[q] = ay[q] = az[q] = 0.f;
        bx[q] = by[q] = bz[q] = 0.f;
        px[q] = py[q] = pz[q] = 0.f;
        dq[q] = i >> 1;
    }
    const int dlo = it.i0 & ~1;
    const int dhi = (iend + 1) & ~1;
    const int jend = it.j0 + it.nj;
    const float crr = e.c.crr;

    for (int t0 = it.j0; t0 < jend; t0 += TJ) {
        const int n = min(TJ, jend - t0);
        float4 A, B;
        float C;
        load_tile_entry(d, t0, jend, t, A, B, C);
        __syncthreads();
        sA[t] = A;
        sB[t] = B;
        sC[t] = C;
        __syncthreads();
        const bool diag = (t0 < dhi) && (t0 + n > dlo);
        /* this wave's part of the tile: the n entries in WJ runs of a
         * multiple of 4 (WJ runs of 4 ceil(n / 4WJ) never pass TJ) */
        const int jw = WJ == 1 ? n : (n + 4 * WJ - 1) / (4 * WJ) * 4;
        const int jb = wj * jw;
        const int nw = max(0, min(jw, n - jb));
        /* Groups of four terms, IPL targets by SU sources (with four sources for
         * every target the shapes of 4 targets per lane took 165 registers in
         * place of 103 to 127). Where the tile holds some of the targets
         * (MASK), what is left over goes source by source, and with steric
         * forces everything, whose registers would cost more waves than the
         * groups gain. Products, us, before and so: 128 spheres 19.9 and 18.6,
         * 8000 with RPY 51.3 and 48.6; 2 targets per lane, four waves, 6000
         * spheres 96.7 and 68.8; 4 targets, one wave, 12000 with RPY 175 and
         * 128. */
        auto sum = [&](auto mask_c) {
            constexpr bool MASK = decltype(mask_c)::value;
            constexpr int SU = 4 / IPL;
            const int n4 = !MASK ? (nw + 3) & ~3 : STERIC ? 0 : nw & ~3;
            for (int jj = jb; jj < jb + n4; jj += 4) {
#pragma unroll
                for (int g = 0; g < 4; g += SU) {
                    const int u0 = jj + g;
                    float4 Aj[SU], Bj[SU];
                    float Fz[SU], rx[4], ry[4], rz[4], ir[4];
#pragma unroll
                    for (int u = 0; u < SU; ++u) {
                        Aj[u] = sA[u0 + u];
                        Bj[u] = sB[u0 + u];
                        Fz[u] = sC[u0 + u];
#pragma unroll
                        for (int q = 0; q < IPL; ++q) {
                            const int p = u * IPL + q;
                            if (SPLIT) {
                                rx[p] = (hx[q] - Aj[u].x) + (lx[q] - Bj[u].x);
                                ry[p] = (hy[q] - Aj[u].y) + (ly[q] - Bj[u].y);
                                rz[p] = (hz[q] - Aj[u].z) + (lz[q] - Bj[u].z);
                            } else {
                                rx[p] = hx[q] - Aj[u].x;
                                ry[p] = hy[q] - Aj[u].y;
                                rz[p] = hz[q] - Aj[u].z;
                            }
                            ir[p] = __builtin_fmaf(rz[p], rz[p], __builtin_fmaf(ry[p], ry[p], rx[p] * rx[p]));
                            /* (the padding past jend may be in reach where lengths are near its 1e15) */
                            if (STERIC && ir[p] < d.list_r2 && ib + q < iend && t0 + u0 + u < jend)
                                append(d.nbr_cnt, d.nbr_idx, &d.ctl->flag, ib + q, t0 + u0 + u);
                        }
                    }
                    rsq4<1>(ir);
#pragma unroll
                    for (int u = 0; u < SU; ++u)
#pragma unroll
                        for (int q = 0; q < IPL; ++q) {
                            const int p = u * IPL + q;
                            if (MASK) ir[p] = (t0 + u0 + u) >> 1 == dq[q] ? 0.f : ir[p];
                            pair_term<RPY>(ir[p], rx[p], ry[p], rz[p], Aj[u].w, Bj[u].w, Fz[u], crr, px[q], py[q],
                                           pz[q]);
                        }
                }
            }
            if (!MASK) return;
            for (int jj = jb + n4; jj < jb + nw; ++jj) {
                const float4 Aj = sA[jj];
                const float4 Bj = sB[jj];
                const float Fz = sC[jj];
                const int dj = (t0 + jj) >> 1;
#pragma unroll
                for (int q = 0; q < IPL; ++q) {
                    float rx, ry, rz;
                    if (SPLIT) {
                        rx = (hx[q] - Aj.x) + (lx[q] - Bj.x);
                        ry = (hy[q] - Aj.y) + (ly[q] - Bj.y);
                        rz = (hz[q] - Aj.z) + (lz[q] - Bj.z);
                    } else {
                        rx = hx[q] - Aj.x;
                        ry = hy[q] - Aj.y;
                        rz = hz[q] - Aj.z;
                    }
                    float r2 = __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
                    if (STERIC && r2 < d.list_r2 && t0 + jj != ib + q && ib + q < iend)
                        append(d.nbr_cnt, d.nbr_idx, &d.ctl->flag, ib + q, t0 + jj);
                    float ir = (dj == dq[q]) ? 0.f : __builtin_amdgcn_rsqf(r2);
                    pair_term<RPY>(ir, rx, ry, rz, Aj.w, Bj.w, Fz, crr, px[q], py[q], pz[q]);
                }
            }
        };
        if (diag)
            sum(std::integral_constant<bool, true>{});
        else
            sum(std::integral_constant<bool, false>{});
        /* TwoSum of the tile partial into (hi, lo) */
#pragma unroll
        for (int q = 0; q < IPL; ++q) {
            two_sum_acc(ax[q], bx[q], px[q]);
            two_sum_acc(ay[q], by[q], py[q]);
            two_sum_acc(az[q], bz[q], pz[q]);
            px[q] = py[q] = pz[q] = 0.f;
        }
    }
    if (WJ > 1) {
        /* combine the WJ waves that share these targets, in wave order */
        __syncthreads(); /* the last tile is no longer read */
        if (wj > 0) {
#pragma unroll
            for (int q = 0; q < IPL; ++q) {
                float* r = lds.red[wj][slot * IPL + q];
                r[0] = ax[q]; r[1] = bx[q]; r[2] = ay[q]; r[3] = by[q]; r[4] = az[q]; r[5] = bz[q];
            }
        }
        __syncthreads();
        if (wj == 0) {
#pragma unroll
            for (int w = 1; w < WJ; ++w) {
#pragma unroll
                for (int q = 0; q < IPL; ++q) {
                    const float* r = lds.red[w][slot * IPL + q];
                    two_sum_acc(ax[q], bx[q], r[0]); bx[q] = bx[q] + r[1];
                    two_sum_acc(ay[q], by[q], r[2]); by[q] = by[q] + r[3];
                    two_sum_acc(az[q], bz[q], r[4]); bz[q] = bz[q] + r[5];
                }
            }
        }
    }
    if (wj == 0) {
        const long long base = d.sys_pbase[it.sys] + (long long)it.c * d.ncomp * it.Nb;
#pragma unroll
        for (int q = 0; q < IPL; ++q) {
            const int i = ib + q;
            if (i < iend) {
                const int li = i - it.ioff;
                d.part[base + li] = (double)ax[q] + (double)bx[q];
                d.part[base + it.Nb + li] = (double)ay[q] + (double)by[q];
                d.part[base + 2 * it.Nb + li] = (double)az[q] + (double)bz[q];
            }
        }
    }
}

/* (hi, lo) += (oh, ol) with TwoSum; the same bits whichever is added to which */
__device__ __forceinline__ void add_hilo(float& hi, float& lo, float oh, float ol) {
    const float s = hi + oh;
    const float bb = s - hi;
    const float err = (hi - (s - bb)) + (oh - bb);
    hi = s;
    lo = (lo + ol) + err;
}

/* The sums v = (hi.x, lo.x, hi.y, lo.y, hi.z, lo.z) of the lanes that agree
 * modulo TI (4, 8 or 16), added up; every lane ends with the total of its
 * class. Distances 8 and 4 by DPP rotations of a row (after the first, rows
 * repeat every 8 lanes, so a rotation by 4 is an exchange at distance 4), 16
 * and 32 by row and half-wave swaps, all VALU operations: no LDS round trip
 * per level. */
template <int TI>
__device__ __forceinline__ void wave_add_hilo(float v[6]) {
    auto ror = [&](auto ctrl) {
        float o[6];
#pragma unroll
        for (int q = 0; q < 6; ++q)
            o[q] = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v[q]),
                                                                      decltype(ctrl)::value, 0xF, 0xF, true));
#pragma unroll
        for (int a = 0; a < 3; ++a) add_hilo(v[2 * a], v[2 * a + 1], o[2 * a], o[2 * a + 1]);
    };
    if (TI <= 8) ror(std::integral_constant<int, 0x128>{}); /* row_ror:8 */
    if (TI <= 4) ror(std::integral_constant<int, 0x124>{}); /* row_ror:4 */
    auto swap = [&](auto rows) {
        float o[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const unsigned x = __builtin_bit_cast(unsigned, v[q]);
            const auto r = decltype(rows)::value == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                                                       : __builtin_amdgcn_permlane32_swap(x, x, false, false);
            /* (a bit cast of the vector's element itself takes element 0) */
            const unsigned r0 = r[0], r1 = r[1];
            v[q] = __builtin_bit_cast(float, r0);
            o[q] = __builtin_bit_cast(float, r1);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) add_hilo(v[2 * a], v[2 * a + 1], o[2 * a], o[2 * a + 1]);
    };
    swap(std::integral_constant<int, 16>{});
    swap(std::integral_constant<int, 32>{});
}

/* ------------------------------------------------------- fused stage */

/* One stage in one kernel. A work-group of NW waves owns FS_I = 16 target
 * spheres of one system and holds all of that system's sources in LDS: lane
 * (wave w, quarter g, target t) sums target t over the sources
 * j = JS m + 4w + g (JS = 4 NW source splits, m = 0, 1, ...) in FP32, with a
 * TwoSum into a (hi, lo) pair every FS_M sources (32 for one system, 64 for
 * an ensemble). The JS partial sums of a target are combined in a fixed order
 * (two shuffles inside the wave, then the NW waves through LDS in a pairwise
 * tree), and wave 0 then does the stage update, next spring forces and next
 * pack of the 8 dumbbells (as the epilogue does, in the rsqrt forms) with no
 * further barrier: a stage needs no partial sums in HBM and no second
 * launch. Only the one term of the
 * JS-source block that holds the work-group's own dumbbells needs the
 * self/partner mask, so only its group of four has it. A single system uses
 * NW = 16 and target blocks in order; an ensemble NW = 4 and a work list of
 * (system, target block), longest system first. The groups' loops are not
 * unrolled further: two groups in flight took 111 registers, four waves per
 * SIMD, and ensembles, whose many small work-groups hide each other's
 * latencies, want the six that 80 registers allow (500 systems of 125 dumbbells
 * 126 us per RK4 step unrolled, 101 not; 64 of 343 82 and 75; one of 1000 35.2 and 35.1). */
constexpr int FS_I = 16;

/* One source entry of the fused stage: sphere t0 + t of the pack, or
 * padding (far away and force-free). With single-float positions only
 * A = (x, y, z, Fx) and C = (Fy, Fz) are read, 24 B per source. */
template <int SPLIT>
__device__ __forceinline__ void load_stage_entry(const Dev& d, int t0, int jend, int t, float4& A, float4& B,
                                                 float& Fy, float& Fz) {
    if (t0 + t < jend) {
        A = d.pA[t0 + t];
        if (SPLIT) {
            B = d.pB[t0 + t];
            Fy = B.w;
            Fz = d.pC[t0 + t].y;
        } else {
            const float2 c = d.pC[t0 + t];
            Fy = c.x;
            Fz = c.y;
        }
    } else {
        A = make_float4(1.0e15f, 1.0e15f, 1.0e15f, 0.f);
        B = make_float4(0.f, 0.f, 0.f, 0.f);
        Fy = 0.f;
        Fz = 0.f;
    }
}

template <int SPLIT, int RPY, int NW>
__global__ __launch_bounds__(64 * NW) void k_stage_fused(Dev d, Epi e) {
    constexpr int T = 64 * NW; /* lanes */
    constexpr int JS = 4 * NW; /* source splits per target */
    /* sources per FP32 partial sum before it is folded into (hi, lo) */
    constexpr int FS_M = NW == 16 ? 32 : 64;
    extern __shared__ float4 fs_lds[];
    const int N = d.Ntot;
    const int tid = threadIdx.x;

    /* the work-group's targets [i0, i0 + ni) in the system [off, off + Nb) */
    int i0, ni, off, Nb;
    if (d.nfitems == 0) {
        i0 = blockIdx.x * FS_I;
        off = 0;
        Nb = N;
    } else {
        const Item it = d.fitems[blockIdx.x];
        i0 = it.i0;
        off = it.ioff;
        Nb = it.Nb;
    }
    ni = min(FS_I, off + Nb - i0);
    const int np = (Nb + JS - 1) / JS * JS;
    /* sources: A = (x, y, z, Fx) [np]; with hi/lo B = (lo.x, lo.y, lo.z, Fy)
     * [np] and Fz [np], else (Fy, Fz) [np] */
    float4* sA = fs_lds;
    float4* sB = fs_lds + np;
    float* sC = reinterpret_cast<float*>(fs_lds + 2 * np);
    float2* sF = reinterpret_cast<float2*>(fs_lds + np);
    const long long step = (e.stage == 0) ? d.ctl->slot[0] : d.ctl->slot[1];
    /* inputs of the closing update, loaded first: lane 3t + a owns
     * component a of target i0 + t */
    double u0 = 0.0, xv = 0.0, rv = 0.0;
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        const int o = a * N + i0 + tt;
        u0 = d.U0[o];
        xv = d.X[o];
        if (e.stage > 0) rv = d.R[o];
    }

    const int w = tid >> 6, l = tid & 63, t = l & 15, g = l >> 4;
    const int js = 4 * w + g;
    const int i = i0 + t;
    /* this lane's target position */
    float hx = 0.f, hy = 0.f, hz = 0.f, lx = 0.f, ly = 0.f, lz = 0.f;
    if (t < ni) {
        const float4 A = d.pA[i];
        hx = A.x; hy = A.y; hz = A.z;
        if (SPLIT) {
            const float4 B = d.pB[i];
            lx = B.x; ly = B.y; lz = B.z;
        }
    }

    /* the system's sources into LDS (padding far away and force-free) */
    for (int j = tid; j < np; j += T) {
        float4 A, B;
        float Fy, Fz;
        load_stage_entry<SPLIT>(d, off, off + Nb, j, A, B, Fy, Fz);
        sA[j] = A;
        if (SPLIT) {
            sB[j] = B;
            sC[j] = Fz;
        } else {
            sF[j] = make_float2(Fy, Fz);
        }
    }
    const int di = (i - off) >> 1; /* local dumbbell (off is even) */
    __syncthreads();
    /* after the staging barrier, in flight under the sums: the step slots for
     * the next kernel, for lane q < ni the phase of dumbbell q/2 and the
     * (sin, cos)(omega t) of this stage, and the noise of the lane's component */
    advance_step(d, e, step);
    double st = 0.0, ct = 0.0, nz = 0.0;
    double2 tp = make_double2(0.0, 0.0);
    if (tid < ni) {
        const long long row = step & (d.ring - 1);
        st = d.tab[row * 8 + 2 * e.stage];
        ct = d.tab[row * 8 + 2 * e.stage + 1];
        tp = d.phitrig[(i0 >> 1) + (tid >> 1)];
    }
    if (e.c.noise && tid < 3 * ni) {
        nz = stage_noise(e.c, i0 + tid / 3, step, tid % 3);
        asm volatile("" : "+v"(nz)); /* formed here, not where the update needs it */
    }

    const float crr = e.c.crr;
    float ax = 0.f, ay = 0.f, az = 0.f, bx = 0.f, by = 0.f, bz = 0.f;
    auto term = [&](int j, bool masked, float& px, float& py, float& pz) {
        const float4 Aj = sA[j];
        float Fy, Fz, qx = 0.f, qy = 0.f, qz = 0.f;
        if (SPLIT) {
            const float4 Bj = sB[j];
            qx = Bj.x; qy = Bj.y; qz = Bj.z;
            Fy = Bj.w;
            Fz = sC[j];
        } else {
            const float2 f = sF[j];
            Fy = f.x;
            Fz = f.y;
        }
        float rx, ry, rz;
        if (SPLIT) {
            rx = (hx - Aj.x) + (lx - qx);
            ry = (hy - Aj.y) + (ly - qy);
            rz = (hz - Aj.z) + (lz - qz);
        } else {
            rx = hx - Aj.x;
            ry = hy - Aj.y;
            rz = hz - Aj.z;
        }
        const float r2 = __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
        float ir = __builtin_amdgcn_rsqf(r2);
        if (masked && (j >> 1) == di) ir = 0.f;
        pair_term<RPY>(ir, rx, ry, rz, Aj.w, Fy, Fz, crr, px, py, pz);
    };
    const Target me{hx, hy, hz, lx, ly, lz};
    auto quad = [&](int x0, auto mask_c, float& px, float& py, float& pz) {
        group_terms<SPLIT, RPY, 1, decltype(mask_c)::value>(me, sA, sB, sC, sF, x0, JS, crr, px, py, pz, di);
    };
    constexpr std::integral_constant<int, 0> plain{};
    constexpr std::integral_constant<int, 1> masked{};
    const int M = np / JS;
    const int ms = (i0 - off) / JS; /* the source block holding this group's dumbbells */
    for (int m0 = 0; m0 < M; m0 += FS_M) {
        const int m1 = min(M, m0 + FS_M);
        float px = 0.f, py = 0.f, pz = 0.f;
        if (ms >= m0 && ms < m1) {
            const int mq = m0 + ((ms - m0) & ~3); /* the group of four that holds ms */
            int m = m0;
#pragma unroll 1
            for (; m < mq; m += 4) quad(js + JS * m, plain, px, py, pz);
            if (m + 4 <= m1) {
                quad(js + JS * m, masked, px, py, pz);
                m += 4;
            }
#pragma unroll 1
            for (; m + 4 <= m1; m += 4) quad(js + JS * m, plain, px, py, pz);
            for (; m < m1; ++m) term(js + JS * m, true, px, py, pz);
        } else if (m1 - m0 == FS_M) {
#pragma unroll 1
            for (int m = m0; m < m0 + FS_M; m += 4) quad(js + JS * m, plain, px, py, pz);
        } else {
            int m = m0;
            for (; m + 4 <= m1; m += 4) quad(js + JS * m, plain, px, py, pz);
            for (; m < m1; ++m) term(js + JS * m, false, px, py, pz);
        }
        two_sum_acc(ax, bx, px);
        two_sum_acc(ay, by, py);
        two_sum_acc(az, bz, pz);
    }

    /* combine the JS partial sums of each target in a fixed order: the four
     * quarters of a wave by shuffles (both partners get the same sum), then
     * the NW waves through LDS in a pairwise tree */
    float v[6] = {ax, bx, ay, by, az, bz};
    wave_add_hilo<16>(v);
    __syncthreads(); /* the sources are no longer read */
    float* red = reinterpret_cast<float*>(fs_lds);                  /* [NW waves][FS_I][6] */
    double* ys = reinterpret_cast<double*>(fs_lds) + NW * FS_I * 3; /* [FS_I][3] stage positions */
    if (g == 0) {
        float* r = red + (w * FS_I + t) * 6;
        for (int q = 0; q < 6; ++q) r[q] = v[q];
    }
    __syncthreads();
    /* wave 0 closes the stage alone */
    if (w != 0) return;
    int bad = 0;
    if (tid < 3 * ni) {
        /* component a of target tt: the waves' sums combined pairwise in a
         * fixed tree (wave w with w + 1, then pairs of pairs, ...), then the
         * stage update */
        const int tt = tid / 3, a = tid - 3 * tt;
        float hs[NW], ls[NW];
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const float* r = red + (ww * FS_I + tt) * 6 + 2 * a;
            hs[ww] = r[0];
            ls[ww] = r[1];
        }
#pragma unroll
        for (int sp = 1; sp < NW; sp *= 2)
#pragma unroll
            for (int ww = 0; ww < NW; ww += 2 * sp) add_hilo(hs[ww], ls[ww], hs[ww + sp], ls[ww + sp]);
        const int ii = i0 + tt;
        const double k = u0 + e.c.co * ((double)hs[0] + (double)ls[0]);
        bad = !isfinite(k);
        ys[tt * 3 + a] = stage_update(d, e, a * N + ii, k, xv, rv, nz);
    }
    /* LDS operations of one wave complete in order: the fences only keep
     * the compiler from moving the reads of ys above its writes */
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (__any(bad) && tid == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (tid < ni) {
        /* one lane per sphere: the spring forces of its dumbbell (both lanes
         * of a dumbbell evaluate the same expression, so they agree bit for
         * bit), then its partner term and its part of the next pack */
        const int q = tid >> 1, h = tid & 1;
        double f[2][3];
        const double id =
            spring_forces_rs(e.c, ys + (2 * q) * 3, ys + (2 * q + 1) * 3, tp.x, tp.y, st, ct, f[0], f[1]);
        store_pack_sphere_rs<SPLIT>(d, e.c, i0 + tid, ys + tid * 3, ys + (tid ^ 1) * 3, f[h], f[h ^ 1], id);
    }
}

/* Wide form of the fused stage, for ensembles of small systems: a work-group
 * of 4 waves owns FW_I = 64 target spheres of one system, one per lane, and
 * holds all of the system's sources in LDS. Wave w sums, for every target,
 * the sources of its quarter [w Q, (w + 1) Q) of the padded source list
 * (Q = np / 4), each read as an LDS broadcast, in FP32 with a TwoSum into
 * (hi, lo) every FW_M sources. Only the sources that are the work-group's own
 * spheres need the self/partner test; they go four at a time too (one at a
 * time, each waiting for its own LDS reads, a work-group waited for the wave
 * that holds them: 128 systems of 16 to 200 dumbbells 51.0 us per RK4 step, 40.8
 * this way; 512 of 16 to 400 229 and 220). The quarters' sums of a target are
 * combined through LDS as (q0 + q1) + (q2 + q3), and the closing update is
 * the one of k_stage_fused. Per work-group, staging and the closing update
 * cost what they cost for 16 targets, over four times the pair work. */
constexpr int FW_M = 32;

template <int SPLIT, int RPY>
__global__ __launch_bounds__(256) void k_stage_wide(Dev d, Epi e) {
    extern __shared__ float4 fs_lds[];
    const int N = d.Ntot;
    const int tid = threadIdx.x;
    const Item it = d.fitems[blockIdx.x];
    const int i0 = it.i0, off = it.ioff, Nb = it.Nb;
    const int ni = min(FW_I, off + Nb - i0);
    const int np = (Nb + 3) / 4 * 4;
    const int Q = np / 4;
    float4* sA = fs_lds;
    float4* sB = fs_lds + np;
    float* sC = reinterpret_cast<float*>(fs_lds + 2 * np);
    float2* sF = reinterpret_cast<float2*>(fs_lds + np);
    const long long step = (e.stage == 0) ? d.ctl->slot[0] : d.ctl->slot[1];
    /* inputs of the closing update, loaded first: lane 3t + a owns
     * component a of target i0 + t */
    double u0 = 0.0, xv = 0.0, rv = 0.0;
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        const int o = a * N + i0 + tt;
        u0 = d.U0[o];
        xv = d.X[o];
        if (e.stage > 0) rv = d.R[o];
    }
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int i = i0 + l;
    /* this lane's target position (lanes past the block's end sum for
     * position zero and are not used) */
    float hx = 0.f, hy = 0.f, hz = 0.f, lx = 0.f, ly = 0.f, lz = 0.f;
    if (l < ni) {
        const float4 A = d.pA[i];
        hx = A.x; hy = A.y; hz = A.z;
        if (SPLIT) {
            const float4 B = d.pB[i];
            lx = B.x; ly = B.y; lz = B.z;
        }
    }
    /* the system's sources into LDS (padding far away and force-free) */
    for (int j = tid; j < np; j += 256) {
        float4 A, B;
        float Fy, Fz;
        load_stage_entry<SPLIT>(d, off, off + Nb, j, A, B, Fy, Fz);
        sA[j] = A;
        if (SPLIT) {
            sB[j] = B;
            sC[j] = Fz;
        } else {
            sF[j] = make_float2(Fy, Fz);
        }
    }
    const int di = (i - off) >> 1; /* local dumbbell (off is even) */
    __syncthreads();
    /* as in k_stage_fused: after the staging barrier */
    advance_step(d, e, step);
    double st = 0.0, ct = 0.0, nz = 0.0;
    double2 tp = make_double2(0.0, 0.0);
    if (tid < ni) {
        const long long row = step & (d.ring - 1);
        st = d.tab[row * 8 + 2 * e.stage];
        ct = d.tab[row * 8 + 2 * e.stage + 1];
        tp = d.phitrig[(i0 >> 1) + (tid >> 1)];
    }
    if (e.c.noise && tid < 3 * ni) {
        nz = stage_noise(e.c, i0 + tid / 3, step, tid % 3);
        asm volatile("" : "+v"(nz)); /* formed here, not where the update needs it */
    }

    const float crr = e.c.crr;
    float ax = 0.f, ay = 0.f, az = 0.f, bx = 0.f, by = 0.f, bz = 0.f;
    auto term = [&](int j, bool masked, float& px, float& py, float& pz) {
        const float4 Aj = sA[j];
        float Fy, Fz, qx = 0.f, qy = 0.f, qz = 0.f;
        if (SPLIT) {
            const float4 Bj = sB[j];
            qx = Bj.x; qy = Bj.y; qz = Bj.z;
            Fy = Bj.w;
            Fz = sC[j];
        } else {
            const float2 f = sF[j];
            Fy = f.x;
            Fz = f.y;
        }
        float rx, ry, rz;
        if (SPLIT) {
            rx = (hx - Aj.x) + (lx - qx);
            ry = (hy - Aj.y) + (ly - qy);
            rz = (hz - Aj.z) + (lz - qz);
        } else {
            rx = hx - Aj.x;
            ry = hy - Aj.y;
            rz = hz - Aj.z;
        }
        const float r2 = __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
        float ir = __builtin_amdgcn_rsqf(r2);
        if (masked && (j >> 1) == di) ir = 0.f;
        pair_term<RPY>(ir, rx, ry, rz, Aj.w, Fy, Fz, crr, px, py, pz);
    };
    const Target me{hx, hy, hz, lx, ly, lz};
    auto quad = [&](int x0, auto mask_c, float& px, float& py, float& pz) {
        group_terms<SPLIT, RPY, 1, decltype(mask_c)::value>(me, sA, sB, sC, sF, x0, 1, crr, px, py, pz, di);
    };
    constexpr std::integral_constant<int, 0> plain{};
    constexpr std::integral_constant<int, 1> masked{};
    /* this wave's quarter of the sources, and the part of it that holds the
     * work-group's own spheres (local [i0 - off, i0 - off + ni)) */
    const int j0 = w * Q, j1 = j0 + Q;
    const int jm0 = max(j0, i0 - off), jm1 = min(j1, i0 - off + ni);
    for (int c0 = j0; c0 < j1; c0 += FW_M) {
        const int c1 = min(j1, c0 + FW_M);
        float px = 0.f, py = 0.f, pz = 0.f;
        if (c0 < jm1 && c1 > jm0) {
            int j = c0;
            for (; j + 4 <= c1; j += 4) quad(j, masked, px, py, pz);
            for (; j < c1; ++j) term(j, true, px, py, pz);
        } else if (c1 - c0 == FW_M) {
            for (int j = c0; j < c0 + FW_M; j += 4) quad(j, plain, px, py, pz);
        } else {
            int j = c0;
            for (; j + 4 <= c1; j += 4) quad(j, plain, px, py, pz);
            for (; j < c1; ++j) term(j, false, px, py, pz);
        }
        two_sum_acc(ax, bx, px);
        two_sum_acc(ay, by, py);
        two_sum_acc(az, bz, pz);
    }

    __syncthreads(); /* the sources are no longer read */
    float* red = reinterpret_cast<float*>(fs_lds);                   /* [4 waves][FW_I][6] */
    double* ys = reinterpret_cast<double*>(fs_lds) + 4 * FW_I * 3;   /* [FW_I][3] stage positions */
    int* badf = reinterpret_cast<int*>(ys + FW_I * 3);
    {
        float* r = red + (w * FW_I + l) * 6;
        r[0] = ax; r[1] = bx; r[2] = ay; r[3] = by; r[4] = az; r[5] = bz;
    }
    if (tid == 0) *badf = 0;
    __syncthreads();
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        float hs[4], ls[4];
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
            const float* r = red + (ww * FW_I + tt) * 6 + 2 * a;
            hs[ww] = r[0];
            ls[ww] = r[1];
        }
        add_hilo(hs[0], ls[0], hs[1], ls[1]);
        add_hilo(hs[2], ls[2], hs[3], ls[3]);
        add_hilo(hs[0], ls[0], hs[2], ls[2]);
        const int ii = i0 + tt;
        const double k = u0 + e.c.co * ((double)hs[0] + (double)ls[0]);
        if (!isfinite(k)) *badf = 1;
        ys[tt * 3 + a] = stage_update(d, e, a * N + ii, k, xv, rv, nz);
    }
    __syncthreads();
    if (tid == 0 && *badf) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (tid < ni) {
        /* one lane per sphere, as in k_stage_fused */
        const int q = tid >> 1, h = tid & 1;
        double f[2][3];
        const double id =
            spring_forces_rs(e.c, ys + (2 * q) * 3, ys + (2 * q + 1) * 3, tp.x, tp.y, st, ct, f[0], f[1]);
        store_pack_sphere_rs<SPLIT>(d, e.c, i0 + tid, ys + tid * 3, ys + (tid ^ 1) * 3, f[h], f[h ^ 1], id);
    }
}

/* Streamed form of the fused stage (ad_launch.fused = 3). The work-group of
 * NW waves owns TI target spheres. TI = 4, 8 or 16 (stream_targets) keeps
 * about one work-group per compute unit: at N = 4096, TI = 8 puts two
 * work-groups on a compute unit and measured 22 % slower, since every
 * work-group reads every source; at N = 2048, TI = 16 leaves half the compute
 * units idle and measured 18 % slower. NW = 16, or 8 with 4 targets
 * (stream_waves): with 8 waves N = 512 ran 16 % faster and N = 1024 9 %, while
 * N = 4096 with 16 targets ran 10 % slower. Each of its source splits
 * (wave w, lane group g of TI lanes) owns a contiguous range of Q sources
 * (Q a multiple of TI). A wave streams its ranges through a double-buffered LDS
 * slot of its own, TI sources per split at a time, one entry per lane: the
 * loads of the chunk after next are in flight while the current chunk is
 * summed (two register sets; 0.5 % off a 4096-sphere step, 1.3 % at 8192), no
 * work-group barrier separates loading from summing, and no system is too
 * large for LDS. Lane (w, g, t) sums target t over its split's range in
 * ascending order, folding into (hi, lo) every 32 sources. LDS ops of one
 * wave complete in order, so the slot needs no barrier: a chunk is written
 * after the wave's reads of the chunk it replaces and read after its own
 * writes. (Interleaving the groups' entries within a slot measured slower.)
 * The partial sums are combined in k_stage_fused's order, through an LDS
 * area beside the slots, so one work-group barrier precedes the closing
 * update; wave 0 then does it alone (stage update, spring forces and pack,
 * in the rsqrt forms) with no further barrier.
 * BAL: with one work-group per compute unit, the waves of a SIMD keep pace:
 * a wave lowers its issue priority one step per quarter of its chunks, so
 * the SIMD issues from the waves that are behind. Under the default oldest-
 * first choice the first waves finish early and the last run with fewer
 * waves to hide their latencies; kept in step, all four waves issue until
 * the end (N = 4096: 7 % off the step). With two work-groups per compute
 * unit the early finishers' closing update overlaps the other work-group's
 * sums instead, and keeping pace was 6 % slower (N = 8192), as it was with
 * fewer chunks per lane (1-3 % at N = 512 and 2048). */
template <int SPLIT, int RPY, int TI, int NW, int BAL, int NOISE>
__device__ __forceinline__ void stage_stream(const Dev& d, const Epi& e) {
    constexpr int G = 64 / TI;    /* lane groups (splits) per wave */
    constexpr int JS = NW * G;    /* source splits */
    constexpr int FOLD = 32 / TI; /* chunks per (hi, lo) fold */
    extern __shared__ float4 fs_lds[];
    const int N = d.Ntot;
    const int tid = threadIdx.x;
    int i0, off, Nb;
    if (d.nfitems == 0) {
        i0 = blockIdx.x * TI;
        off = 0;
        Nb = N;
    } else {
        const Item it = d.fitems[blockIdx.x];
        i0 = it.i0;
        off = it.ioff;
        Nb = it.Nb;
    }
    const int ni = min(TI, off + Nb - i0);
    const int Q = (Nb + JS * TI - 1) / (JS * TI) * TI; /* sources per split */
    const int K = Q / TI;                              /* chunks per split */
    /* per wave and buffer 64 entries: A = (x, y, z, Fx); with hi/lo
     * B = (lo.xyz, Fy) and Fz, else (Fy, Fz) */
    float4* sA = fs_lds;
    float4* sB = fs_lds + NW * 128;
    float* sC = reinterpret_cast<float*>(fs_lds + 2 * NW * 128);
    float2* sF = reinterpret_cast<float2*>(fs_lds + NW * 128);
    const long long step = (e.stage == 0) ? d.ctl->slot[0] : d.ctl->slot[1];
    /* inputs of the closing update, loaded first */
    double u0 = 0.0, xv = 0.0, rv = 0.0;
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        const int o = a * N + i0 + tt;
        u0 = d.U0[o];
        xv = d.X[o];
        if (e.stage > 0) rv = d.R[o];
    }
    const int w = tid >> 6, l = tid & 63, t = l % TI, g = l / TI;
    const int sp = G * w + g; /* this lane's source split */
    const int i = i0 + t;
    float hx = 0.f, hy = 0.f, hz = 0.f, lx = 0.f, ly = 0.f, lz = 0.f;
    if (t < ni) {
        const float4 A = d.pA[i];
        hx = A.x; hy = A.y; hz = A.z;
        if (SPLIT) {
            const float4 B = d.pB[i];
            lx = B.x; ly = B.y; lz = B.z;
        }
    }
    const int di = (i - off) >> 1;
    /* the chunk holding the work-group's own spheres: split so, chunk ko */
    const int so = (i0 - off) / Q, ko = ((i0 - off) - so * Q) / TI;
    const bool own_wave = so / G == w;

    /* two register sets: chunk k + 2 is loaded while chunk k is summed */
    float4 eA0, eB0, eA1, eB1;
    float eFy0, eFz0, eFy1, eFz1;
    auto fetch = [&](int k, auto R) {
        if constexpr (decltype(R)::value == 0)
            load_stage_entry<SPLIT>(d, off, off + Nb, sp * Q + k * TI + t, eA0, eB0, eFy0, eFz0);
        else
            load_stage_entry<SPLIT>(d, off, off + Nb, sp * Q + k * TI + t, eA1, eB1, eFy1, eFz1);
    };
    auto put = [&](int buf, auto R) {
        constexpr int r = decltype(R)::value;
        const int x = (w * 2 + buf) * 64 + g * TI + t;
        sA[x] = r ? eA1 : eA0;
        if (SPLIT) {
            sB[x] = r ? eB1 : eB0;
            sC[x] = r ? eFz1 : eFz0;
        } else {
            sF[x] = r ? make_float2(eFy1, eFz1) : make_float2(eFy0, eFz0);
        }
    };
    fetch(0, std::integral_constant<int, 0>{});
    /* With few sources per lane (4 or 8 targets) wave 0, which closes the
     * stage, is what the work-group waits for: it reads the step index, issues
     * the loads that depend on it and forms the noise while its first sources
     * arrive. With 16 targets its sums are not the last to finish: sources go
     * first, and the noise, whose code in front of the sums cost 1 to 2 % at
     * N = 6000 and 8192 even unused, is formed at the update. */
    if (TI == 16) put(0, std::integral_constant<int, 0>{});
    if (K > 1) fetch(1, std::integral_constant<int, 1>{});
    advance_step(d, e, step);
    double st = 0.0, ct = 0.0, nz = 0.0;
    double2 tp = make_double2(0.0, 0.0);
    if (tid < ni) {
        const long long row = step & (d.ring - 1);
        st = d.tab[row * 8 + 2 * e.stage];
        ct = d.tab[row * 8 + 2 * e.stage + 1];
        tp = d.phitrig[(i0 >> 1) + (tid >> 1)];
    }
    if (NOISE && TI < 16 && tid < 3 * ni) {
        nz = stage_noise(e.c, i0 + tid / 3, step, tid % 3);
        asm volatile("" : "+v"(nz)); /* formed here, not where the update needs it */
    }
    if (TI < 16) put(0, std::integral_constant<int, 0>{});

    const float crr = e.c.crr;
    float ax = 0.f, ay = 0.f, az = 0.f, bx = 0.f, by = 0.f, bz = 0.f;
    auto term = [&](int x, int j, bool masked, float& px, float& py, float& pz) {
        const float4 Aj = sA[x];
        float Fy, Fz, qx = 0.f, qy = 0.f, qz = 0.f;
        if (SPLIT) {
            const float4 Bj = sB[x];
            qx = Bj.x; qy = Bj.y; qz = Bj.z;
            Fy = Bj.w;
            Fz = sC[x];
        } else {
            const float2 f = sF[x];
            Fy = f.x;
            Fz = f.y;
        }
        float rx, ry, rz;
        if (SPLIT) {
            rx = (hx - Aj.x) + (lx - qx);
            ry = (hy - Aj.y) + (ly - qy);
            rz = (hz - Aj.z) + (lz - qz);
        } else {
            rx = hx - Aj.x;
            ry = hy - Aj.y;
            rz = hz - Aj.z;
        }
        const float r2 = __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
        float ir = BAL ? __builtin_amdgcn_rsqf(r2) : rsq1(r2);
        if (masked && (j >> 1) == di) ir = 0.f;
        pair_term<RPY>(ir, rx, ry, rz, Aj.w, Fy, Fz, crr, px, py, pz);
    };
    const Target me{hx, hy, hz, lx, ly, lz};
    /* terms per group: two with hi/lo positions and 8 targets, where groups of
     * four took 128 to 131 registers and with RPY or noise left a compute unit
     * one work-group (3072 spheres, RPY, us per RK4 step: 63.5, 54.8 this way; a
     * cap at 128 spills, 56.8, and 27.2 against 28.4 at 1400) */
    constexpr int NT = SPLIT && TI == 8 ? 2 : 4;
    auto group = [&](int x0, float& px, float& py, float& pz) {
        group_terms<SPLIT, RPY, !BAL, 0, NT>(me, sA, sB, sC, sF, x0, 1, crr, px, py, pz);
    };
    float px = 0.f, py = 0.f, pz = 0.f;
    auto chunk = [&](int k, auto R) {
        constexpr int r = decltype(R)::value; /* = k & 1, the buffer and the set of chunk k */
        if (BAL) {
            const int lvl = (4 * k) / K;
            if (lvl == 0) __builtin_amdgcn_s_setprio(3);
            else if (lvl == 1) __builtin_amdgcn_s_setprio(2);
            else if (lvl == 2) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        if (k + 2 < K) fetch(k + 2, R);
        const int x0 = (w * 2 + r) * 64 + g * TI;
        const int j0 = sp * Q + k * TI;
        if (own_wave && k == ko) {
            for (int v = 0; v < TI; ++v) term(x0 + v, j0 + v, true, px, py, pz);
        } else {
            if (TI == 16 && !BAL) {
#pragma unroll
                for (int v = 0; v < TI; ++v) term(x0 + v, j0 + v, false, px, py, pz);
            } else {
#pragma unroll
                for (int v = 0; v < TI; v += NT) group(x0 + v, px, py, pz);
            }
        }
        if ((k + 1) % FOLD == 0 || k + 1 == K) {
            two_sum_acc(ax, bx, px);
            two_sum_acc(ay, by, py);
            two_sum_acc(az, bz, pz);
            px = py = pz = 0.f;
        }
        if (k + 1 < K) put(1 - r, std::integral_constant<int, 1 - r>{});
    };
    for (int k = 0; k < K; k += 2) {
        chunk(k, std::integral_constant<int, 0>{});
        if (k + 1 < K) chunk(k + 1, std::integral_constant<int, 1>{});
    }

    /* combine the partial sums of each target as k_stage_fused does: the G
     * groups of a wave by shuffles, then the waves through LDS in a tree */
    float v[6] = {ax, bx, ay, by, az, bz};
    if (TI == 16) {
        /* sixteen waves keep the VALU busy: the exchanges go through the LDS
         * crossbar instead (VALU swaps 1 % slower at N = 4096 and 8192; with 4
         * or 8 targets the round trips' latency counts, 3 % at N = 512) */
#pragma unroll
        for (int sh = 16; sh < 64; sh *= 2) {
            float o[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) o[q] = __shfl_xor(v[q], sh);
#pragma unroll
            for (int a = 0; a < 3; ++a) add_hilo(v[2 * a], v[2 * a + 1], o[2 * a], o[2 * a + 1]);
        }
    } else {
        wave_add_hilo<TI>(v);
    }
    /* the combination area lies beside the source slots, so no barrier
     * waits for the slowest wave's last reads before it is written */
    float* red = reinterpret_cast<float*>(reinterpret_cast<char*>(fs_lds) + NW * 128 * (SPLIT ? 36 : 24));
    double* ys = reinterpret_cast<double*>(red + NW * TI * 6); /* [TI][3] stage positions */
    if (g == 0) {
        float* r = red + (w * TI + t) * 6;
        for (int q = 0; q < 6; ++q) r[q] = v[q];
    }
    __syncthreads();
    /* wave 0 closes the stage alone */
    if (w != 0) return;
    if (BAL) __builtin_amdgcn_s_setprio(3);
    int bad = 0;
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        float hs[NW], ls[NW];
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const float* r = red + (ww * TI + tt) * 6 + 2 * a;
            hs[ww] = r[0];
            ls[ww] = r[1];
        }
#pragma unroll
        for (int st2 = 1; st2 < NW; st2 *= 2)
#pragma unroll
            for (int ww = 0; ww < NW; ww += 2 * st2) add_hilo(hs[ww], ls[ww], hs[ww + st2], ls[ww + st2]);
        const int ii = i0 + tt;
        const double k = u0 + e.c.co * ((double)hs[0] + (double)ls[0]);
        bad = !isfinite(k);
        if (NOISE && TI == 16) nz = stage_noise(e.c, ii, step, a);
        ys[tt * 3 + a] = stage_update(d, e, a * N + ii, k, xv, rv, nz);
    }
    /* LDS operations of one wave complete in order: the fences only keep
     * the compiler from moving the reads of ys above its writes */
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (__any(bad) && tid == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (tid < ni) {
        const int q = tid >> 1, h = tid & 1;
        double f[2][3];
        const double id =
            spring_forces_rs(e.c, ys + (2 * q) * 3, ys + (2 * q + 1) * 3, tp.x, tp.y, st, ct, f[0], f[1]);
        store_pack_sphere_rs<SPLIT>(d, e.c, i0 + tid, ys + tid * 3, ys + (tid ^ 1) * 3, f[h], f[h ^ 1], id);
    }
}

/* NOISE apart: its registers would not fit beside the others' in the capped
 * instance below (11 spilled, 4 % at N = 8192 without noise) */
template <int SPLIT, int RPY, int TI, int NW, int NOISE>
__global__ __launch_bounds__(64 * NW) void k_stage_stream(Dev d, Epi e) {
    stage_stream<SPLIT, RPY, TI, NW, TI == 16 && NW == 16, NOISE>(d, e);
}

/* The same with registers capped for 8 waves per SIMD (63 VGPRs), so that two
 * 16-wave work-groups share a compute unit: for launches of more than 256
 * work-groups (N = 8192: 4 % faster per step; with one work-group per compute
 * unit, N = 4096, the cap cost 5 %). */
template <int SPLIT, int RPY, int TI, int NW, int NOISE>
__global__ __launch_bounds__(64 * NW, 8) void k_stage_stream_x2(Dev d, Epi e) {
    stage_stream<SPLIT, RPY, TI, NW, 0, NOISE>(d, e);
}

/* FP64 streamed form of the fused stage (AD_FP64_TILED with
 * ad_launch.fused = 3): k_stage_stream's work-group shape, streaming and
 * combination order in FP64 arithmetic, for a like-for-like comparison with
 * the FP32C form. The pair term uses a refined v_rsq_f64 and FMAs (not the
 * IEEE sqrt and divisions of the plain sum); the partial sums are plain FP64 sums. As in the other
 * FP64 forms, the pair sum includes the dumbbell partner and only the self
 * term is masked, u0 is the self term alone, and the pack is the FP64 one
 * (3 double2 per sphere). */
template <int RPY>
__device__ __forceinline__ void pair_term64(double ir, double rx, double ry, double rz, double Fx, double Fy,
                                            double Fz, double crr, double& px, double& py, double& pz) {
    const double fr = __builtin_fma(rz, Fz, __builtin_fma(ry, Fy, rx * Fx));
    const double ir2 = ir * ir;
    const double tt = fr * ir2;
    if (RPY) {
        const double ir3 = ir * ir2;
        const double av = __builtin_fma(crr, ir3, ir);
        const double bv = tt * __builtin_fma(-3.0 * crr, ir3, ir);
        px = __builtin_fma(av, Fx, __builtin_fma(bv, rx, px));
        py = __builtin_fma(av, Fy, __builtin_fma(bv, ry, py));
        pz = __builtin_fma(av, Fz, __builtin_fma(bv, rz, pz));
    } else {
        px = __builtin_fma(ir, __builtin_fma(tt, rx, Fx), px);
        py = __builtin_fma(ir, __builtin_fma(tt, ry, Fy), py);
        pz = __builtin_fma(ir, __builtin_fma(tt, rz, Fz), pz);
    }
}

template <int RPY, int TI>
__global__ __launch_bounds__(1024) void k_stage_stream64(Dev d, Epi e) {
    constexpr int NW = 16;
    constexpr int G = 64 / TI;  /* lane groups (splits) per wave */
    constexpr int JS = NW * G;  /* source splits */
    extern __shared__ double4 fs64_lds[];
    const int N = d.Ntot;
    const int tid = threadIdx.x;
    int i0, off, Nb;
    if (d.nfitems == 0) {
        i0 = blockIdx.x * TI;
        off = 0;
        Nb = N;
    } else {
        const Item it = d.fitems[blockIdx.x];
        i0 = it.i0;
        off = it.ioff;
        Nb = it.Nb;
    }
    const int ni = min(TI, off + Nb - i0);
    const int Q = (Nb + JS * TI - 1) / (JS * TI) * TI; /* sources per split */
    const int K = Q / TI;                              /* chunks per split */
    /* per wave and buffer 64 entries: A = (x, y, z, Fx), F = (Fy, Fz) */
    double4* sA = fs64_lds;
    double2* sF = reinterpret_cast<double2*>(fs64_lds + NW * 128);
    const long long step = (e.stage == 0) ? d.ctl->slot[0] : d.ctl->slot[1];
    double u0 = 0.0, xv = 0.0, rv = 0.0;
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        const int o = a * N + i0 + tt;
        u0 = d.U0[o];
        xv = d.X[o];
        if (e.stage > 0) rv = d.R[o];
    }
    const int w = tid >> 6, l = tid & 63, t = l % TI, g = l / TI;
    const int sp = G * w + g;
    const int i = i0 + t;
    double hx = 0.0, hy = 0.0, hz = 0.0;
    if (t < ni) {
        const double2 a0 = d.pD[3 * i], a1 = d.pD[3 * i + 1];
        hx = a0.x; hy = a0.y; hz = a1.x;
    }
    const int so = (i0 - off) / Q, ko = ((i0 - off) - so * Q) / TI;
    const bool own_wave = so / G == w;

    double4 eA;
    double2 eF;
    auto fetch = [&](int k) {
        const int j = sp * Q + k * TI + t;
        if (off + j < off + Nb) {
            const double2 a0 = d.pD[3 * (off + j)], a1 = d.pD[3 * (off + j) + 1], a2 = d.pD[3 * (off + j) + 2];
            eA = make_double4(a0.x, a0.y, a1.x, a1.y);
            eF = a2;
        } else {
            eA = make_double4(1.0e15, 1.0e15, 1.0e15, 0.0);
            eF = make_double2(0.0, 0.0);
        }
    };
    auto put = [&](int buf) {
        const int x = (w * 2 + buf) * 64 + g * TI + t;
        sA[x] = eA;
        sF[x] = eF;
    };
    fetch(0);
    advance_step(d, e, step);
    double st = 0.0, ct = 0.0, nz = 0.0;
    double2 tp = make_double2(0.0, 0.0);
    if (tid < ni) {
        const long long row = step & (d.ring - 1);
        st = d.tab[row * 8 + 2 * e.stage];
        ct = d.tab[row * 8 + 2 * e.stage + 1];
        tp = d.phitrig[(i0 >> 1) + (tid >> 1)];
    }
    if (e.c.noise && tid < 3 * ni) {
        nz = stage_noise(e.c, i0 + tid / 3, step, tid % 3);
        asm volatile("" : "+v"(nz)); /* formed here, not where the update needs it */
    }
    put(0);

    const double crr = e.c.crr64;
    double px = 0.0, py = 0.0, pz = 0.0;
    auto term = [&](int x, int j, bool masked) {
        const double4 Aj = sA[x];
        const double2 Fj = sF[x];
        const double rx = hx - Aj.x, ry = hy - Aj.y, rz = hz - Aj.z;
        const double r2 = __builtin_fma(rz, rz, __builtin_fma(ry, ry, rx * rx));
        double ir = rsqrt64(r2);
        if (masked && j == i - off) ir = 0.0;
        pair_term64<RPY>(ir, rx, ry, rz, Aj.w, Fj.x, Fj.y, crr, px, py, pz);
    };
    for (int k = 0; k < K; ++k) {
        const int buf = k & 1;
        if (TI == 16) {
            /* the waves of a SIMD keep pace, as in k_stage_stream's
             * one-work-group-per-unit instance (one 16-wave work-group per
             * compute unit fits at this kernel's register count) */
            const int lvl = (4 * k) / K;
            if (lvl == 0) __builtin_amdgcn_s_setprio(3);
            else if (lvl == 1) __builtin_amdgcn_s_setprio(2);
            else if (lvl == 2) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        if (k + 1 < K) fetch(k + 1);
        const int x0 = (w * 2 + buf) * 64 + g * TI;
        const int j0 = sp * Q + k * TI;
        if (own_wave && k == ko) {
            for (int v = 0; v < TI; ++v) term(x0 + v, j0 + v, true);
        } else {
#pragma unroll
            for (int v = 0; v < TI; ++v) term(x0 + v, j0 + v, false);
        }
        if (k + 1 < K) put(buf ^ 1);
    }
    /* the G groups of a wave by shuffles, then the waves through LDS in a
     * pairwise tree: a fixed order */
#pragma unroll
    for (int sh = TI; sh < 64; sh *= 2) {
        px = px + __shfl_xor(px, sh);
        py = py + __shfl_xor(py, sh);
        pz = pz + __shfl_xor(pz, sh);
    }
    double* red = reinterpret_cast<double*>(fs64_lds + NW * 128 + NW * 128 / 2); /* [NW][TI][3] */
    double* ys = red + NW * TI * 3;                                              /* [TI][3] */
    if (g == 0) {
        double* r = red + (w * TI + t) * 3;
        r[0] = px; r[1] = py; r[2] = pz;
    }
    __syncthreads();
    if (w != 0) return;
    if (TI == 16) __builtin_amdgcn_s_setprio(3);
    int bad = 0;
    if (tid < 3 * ni) {
        const int tt = tid / 3, a = tid - 3 * tt;
        double hs[NW];
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) hs[ww] = red[(ww * TI + tt) * 3 + a];
#pragma unroll
        for (int st2 = 1; st2 < NW; st2 *= 2)
#pragma unroll
            for (int ww = 0; ww < NW; ww += 2 * st2) hs[ww] = hs[ww] + hs[ww + st2];
        const int ii = i0 + tt;
        const double k = u0 + e.c.co * hs[0];
        bad = !isfinite(k);
        ys[tt * 3 + a] = stage_update(d, e, a * N + ii, k, xv, rv, nz);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (__any(bad) && tid == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (tid < ni) {
        const int q = tid >> 1, h = tid & 1;
        double f[2][3];
        spring_forces_rs(e.c, ys + (2 * q) * 3, ys + (2 * q + 1) * 3, tp.x, tp.y, st, ct, f[0], f[1]);
        const double* y = ys + tid * 3;
        const int ii = i0 + tid;
        for (int a = 0; a < 3; ++a) d.U0[a * N + ii] = e.c.cs * f[h][a];
        d.pD2[3 * ii + 0] = make_double2(y[0], y[1]);
        d.pD2[3 * ii + 1] = make_double2(y[2], f[h][0]);
        d.pD2[3 * ii + 2] = make_double2(f[h][1], f[h][2]);
    }
}

/* The correctly rounded FP64 quotients of a pair term, sharing work between
 * them: s = sqrt(r2), ir = 1/s, t = fr/r2 and (RPY) ir/r2, each bit for bit
 * the IEEE result of the plain expression.
 *   s: v_rsq_f64 (about 2^-24) refined on g = sqrt(x) and h = 1/(2 sqrt(x)),
 *     then corrected twice by its exact residual x - g^2;
 *   1/s starts from 2h (already within 2^-46) in place of a v_rcp_f64 and a
 *     first Newton step: one step, then the correction by the exact residual
 *     1 - s y, after which the quotient is the rounded one (Markstein, "Computation
 *     of elementary functions on the IBM RISC System/6000 processor", 1990)
 *     unless the divisor's significand is all ones;
 *   1/r2 starts from (2h)^2: one Newton step, then the quotient a y corrected
 *     once by its residual a - r2 q, rounded under the same condition on r2 if
 *     y is the rounded 1/r2.
 * y could be another one only where 1/r2 lies within the step's error (2^-88.8
 * for a v_rsq_f64 anywhere within 2^-23) of a midpoint, and a quotient next to a
 * midpoint goes wrong by that only for significands 2 - 2t of r2 with t < 2^-36
 * (for others |r| |y - 1/r2| stays below every quotient's distance from a
 * midpoint). There 1/r2 is t^2 from the midpoint 1 + t: what remains are the 195
 * significands 2 - (2k + 1) 2^-52. This chip's v_rsq_f64 is within 2^-26.1 there
 * (2^-24.1 elsewhere), and of them y is another one for k = 0, left out, and in
 * one parity k = 1, of which no quotient is that near. (The tests take every k
 * below 260 with its nearest quotients, and emulate the rest with other seeds;
 * the compiler's division fails some of them.)
 * 20 FP64 instructions and one transcendental in place of the compiler's 39
 * and three for the same three values (its square root and divisions also
 * scale the exponents and fix up special operands), and a dependent chain of
 * 15 for both quotients. They hold where no intermediate can leave the normal
 * range: r2 in [2^-400, 2^400) and |fr| zero or in [2^-500, 2^500), and where
 * neither s nor r2 has an all-ones low word; the callers test that (Range64)
 * and take the plain expressions otherwise. */
__device__ __forceinline__ unsigned lo_word(double x) {
    return (unsigned)__builtin_bit_cast(unsigned long long, x);
}
__device__ __forceinline__ unsigned hi_word(double x) {
    return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32);
}
/* The range test over a lane's terms, on high words with 32-bit min and max
 * (an FP64 compare with its select measured 48 cycles per wave, a 32-bit
 * min or max 4): r2 in [2^-400, 2^400) (it is a sum of squares, so its sign
 * bit is clear unless it is NaN, whose high word is larger), |fr| in
 * [2^-500, 2^500), no all-ones low word of s or r2. A zero fr, which needs
 * nothing, counts as too small: zeros() tells it apart. */
struct Range64 {
    unsigned rmin = 0xffffffffu, rmax = 0, fmin = 0xffffffffu, fmax = 0, ones = 0;
    static constexpr unsigned kR2Lo = (1023u - 400u) << 20, kR2Hi = (1023u + 400u) << 20;
    static constexpr unsigned kFrLo = (1023u - 500u) << 21, kFrHi = (1023u + 500u) << 21;
    __device__ __forceinline__ void r2(double x) {
        rmin = min(rmin, hi_word(x));
        rmax = max(rmax, hi_word(x));
    }
    __device__ __forceinline__ void fr(double x) {
        const unsigned h = hi_word(x) << 1; /* without the sign */
        fmin = min(fmin, h);
        fmax = max(fmax, h);
    }
    __device__ __forceinline__ bool ok_r2() const { return rmin >= kR2Lo && rmax < kR2Hi; }
    __device__ __forceinline__ bool ok() const { return ok_r2() && fmax < kFrHi && ones != 0xffffffffu; }
    __device__ __forceinline__ bool small_fr() const { return fmin < kFrLo; }
    /* zero, or not too small */
    static __device__ __forceinline__ bool fr_fits(double x) {
        const unsigned h = hi_word(x) << 1;
        return (h | lo_word(x)) == 0 || h >= kFrLo;
    }
};
/* s = sqrt(x) and ir = 1/s as the plain expressions round them, and y = 1/x
 * (rounded where ones allows the short forms) for div_exact; ones is raised to
 * the low words of s and x */
__device__ __forceinline__ void rcp_sqrt_exact(double x, double& s, double& ir, double& y, unsigned& ones) {
    const double v = __builtin_amdgcn_rsq(x);
    double g = x * v;
    double h = v * 0.5;
    double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    double q = __builtin_fma(-g, g, x);
    g = __builtin_fma(q, h, g);
    q = __builtin_fma(-g, g, x);
    s = __builtin_fma(q, h, g);
    ones = max(ones, max(lo_word(s), lo_word(x)));
    const double h2 = h + h;
    y = h2 * h2;
    y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
    ir = __builtin_fma(h2, __builtin_fma(-s, h2, 1.0), h2);
    ir = __builtin_fma(ir, __builtin_fma(-s, ir, 1.0), ir);
}
/* a/x as IEEE division rounds it, y from rcp_sqrt_exact */
__device__ __forceinline__ double div_exact(double a, double x, double y) {
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-x, q, a), y, q);
}

/* FP64: the sum in ascending j with the plain operation order
 *   r2 = (rx*rx + ry*ry) + rz*rz; ir = 1/sqrt(r2); fr = (rx*Fx + ry*Fy) + rz*Fz;
 *   t = fr/r2; acc = acc + ir*(F + t*r)
 * over every j != i of the chunk (partner included). A coincident pair is
 * skipped and raises the flag. With one chunk per system this is the
 * sequential FP64 sum exactly: AD_FP64 where k_pairs_f64w, which gives the
 * same bits, has no work list. With RPY the correction (F - 3 t r) ir/r2 is
 * summed in a second accumulator. */
template <int WG, int IPL, int RPY>
__global__ __launch_bounds__(WG) void k_pairs_f64(Dev d, Epi e, int mode) {
    __shared__ double2 sD[3][WG];
    const Item it = d.items[blockIdx.x];
    if (mode) advance_slots(d, e);
    const int t = threadIdx.x;
    const int ib = it.i0 + t * IPL;
    const int iend = it.i0 + it.ni;
    double xi[IPL], yi[IPL], zi[IPL], ax[IPL], ay[IPL], az[IPL], bx[IPL], by[IPL], bz[IPL];
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        const int i = ib + q;
        double2 p0 = make_double2(0.0, 0.0), p1 = p0;
        if (i < iend) {
            p0 = d.pD[3 * i];
            p1 = d.pD[3 * i + 1];
        }
        xi[q] = p0.x; yi[q] = p0.y; zi[q] = p1.x;
        ax[q] = ay[q] = az[q] = 0.0;
        bx[q] = by[q] = bz[q] = 0.0;
    }
    int bad = 0;
    const int jend = it.j0 + it.nj;
    for (int t0 = it.j0; t0 < jend; t0 += WG) {
        const int n = min(WG, jend - t0);
        double2 a0, a1, a2;
        if (t < n) {
            a0 = d.pD[3 * (t0 + t)];
            a1 = d.pD[3 * (t0 + t) + 1];
            a2 = d.pD[3 * (t0 + t) + 2];
        } else {
            a0 = make_double2(1.0e300, 1.0e300);
            a1 = make_double2(1.0e300, 0.0);
            a2 = make_double2(0.0, 0.0);
        }
        __syncthreads();
        sD[0][t] = a0;
        sD[1][t] = a1;
        sD[2][t] = a2;
        __syncthreads();
        /* four sources at a time: their terms' square roots and divisions
         * overlap, the additions stay in ascending j (6 % faster than one at
         * a time, 8 at a time 2 %) */
#pragma unroll 4
        for (int jj = 0; jj < n; ++jj) {
            const double2 b0 = sD[0][jj], b1 = sD[1][jj], b2 = sD[2][jj];
            const double Fx = b1.y, Fy = b2.x, Fz = b2.y;
            const int j = t0 + jj;
#pragma unroll
            for (int q = 0; q < IPL; ++q) {
                double rx = xi[q] - b0.x;
                double ry = yi[q] - b0.y;
                double rz = zi[q] - b1.x;
                double r2 = (rx * rx + ry * ry) + rz * rz;
                bool self = (j == ib + q);
                bool skip = self || (r2 == 0.0);
                bad |= (!self && r2 == 0.0);
                double r2s = skip ? 1.0 : r2;
                double ir = 1.0 / sqrt(r2s);
                double fr = (rx * Fx + ry * Fy) + rz * Fz;
                double tt = fr / r2s;
                double gx = ir * (Fx + tt * rx);
                double gy = ir * (Fy + tt * ry);
                double gz = ir * (Fz + tt * rz);
                ax[q] = skip ? ax[q] : ax[q] + gx;
                ay[q] = skip ? ay[q] : ay[q] + gy;
                az[q] = skip ? az[q] : az[q] + gz;
                if (RPY) {
                    const double ir3 = ir / r2s;
                    const double t3 = 3.0 * tt;
                    const double hx = ir3 * (Fx - t3 * rx);
                    const double hy = ir3 * (Fy - t3 * ry);
                    const double hz = ir3 * (Fz - t3 * rz);
                    bx[q] = skip ? bx[q] : bx[q] + hx;
                    by[q] = skip ? by[q] : by[q] + hy;
                    bz[q] = skip ? bz[q] : bz[q] + hz;
                }
            }
        }
    }
    const long long base = d.sys_pbase[it.sys] + (long long)it.c * d.ncomp * it.Nb;
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        const int i = ib + q;
        if (i < iend) {
            const int li = i - it.ioff;
            d.part[base + li] = ax[q];
            d.part[base + it.Nb + li] = ay[q];
            d.part[base + 2 * it.Nb + li] = az[q];
            if (RPY) {
                d.part[base + 3 * it.Nb + li] = bx[q];
                d.part[base + 4 * it.Nb + li] = by[q];
                d.part[base + 5 * it.Nb + li] = bz[q];
            }
            if (bad) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
        }
    }
}

/* AD_FP64_TILED: the sum over every j != i of the chunk (partner included) in
 * FP64 with rsqrt64 and FMAs. A work-group of G waves takes 64 IPL targets of
 * a work item (IPL per lane; an item of more targets is several work-groups)
 * and stages tiles of 64 G sources through LDS; wave w sums the w-th 64 of
 * every tile, F64_J sources at a time, and the waves' sums are added in wave
 * order through LDS. A coincident pair is skipped and raises the flag. Sources
 * whose r2 leaves the range of the short forms for some lane take the plain
 * expressions. With RPY the correction is summed apart.
 * What bounds it is FP64 issue: 23 instructions per term (31 with RPY) beside
 * the range test, against about 60 (70) for the plain form's square root and
 * divisions, which it replaced. A term's error does not grow: root mean
 * square over random pairs, against 128 bits, 1.15e-16 (the FMA into the sum
 * included) against 1.19e-16, and whole products at 100 to 3000 spheres lie
 * 1 to 6 % nearer to 80-bit sums than the plain form's.
 * The split by G waves is for balance and for small systems: one wave per 64
 * targets summing whole chunks left 16 waves on the chip at 512 spheres.
 * One product (pack, this, epilogue), us, against the plain form's: 512
 * spheres 18.3 (60.2), 4096 31 (67), 16384 281 (667); RPY 18.8 (70), 41.5 (85),
 * 357 (888). Two, eight and sixteen waves: 24, 18.3, 19 at 512, 289, 283, 314
 * at 16384. */
constexpr int F64_J = 4;

template <int G, int IPL, int RPY>
__global__ __launch_bounds__(64 * G) void k_pairs_f64t(Dev d, Epi e, int mode, int per_item) {
    constexpr int TJ = 64 * G;
    constexpr int NC = RPY ? 6 : 3;
    union Lds {
        double2 src[3][TJ];
        double red[G > 1 ? G - 1 : 1][NC * IPL][64];
    };
    __shared__ Lds lds;
    if (mode) advance_slots(d, e);
    const Item it = d.items[blockIdx.x / per_item];
    const int t = threadIdx.x, l = t & 63, w = t >> 6;
    const int b0 = it.i0 + (int)(blockIdx.x % per_item) * 64 * IPL; /* first target of the group */
    const int iend = it.i0 + it.ni;
    if (b0 >= iend) return;
    const int bend = min(iend, b0 + 64 * IPL);
    const int ib = b0 + l * IPL;
    double xi[IPL], yi[IPL], zi[IPL], acc[IPL][6];
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        const int i = min(ib + q, bend - 1); /* lanes past the end repeat the last target, unused */
        const double2 p0 = d.pD[3 * i], p1 = d.pD[3 * i + 1];
        xi[q] = p0.x; yi[q] = p0.y; zi[q] = p1.x;
#pragma unroll
        for (int c = 0; c < 6; ++c) acc[q][c] = 0.0;
    }
    int bad = 0;
    const int jend = it.j0 + it.nj;
    for (int t0 = it.j0; t0 < jend; t0 += TJ) {
        const int j = min(t0 + t, jend - 1);
        const double2 a0 = d.pD[3 * j], a1 = d.pD[3 * j + 1], a2 = d.pD[3 * j + 2];
        __syncthreads();
        lds.src[0][t] = a0;
        lds.src[1][t] = a1;
        lds.src[2][t] = a2;
        __syncthreads();
        const int n = min(64, jend - t0 - 64 * w); /* this wave's sources of the tile */
        auto plain = [&](int jj) {
            const double2 c0 = lds.src[0][jj], c1 = lds.src[1][jj], c2 = lds.src[2][jj];
            const double F[3] = {c1.y, c2.x, c2.y};
#pragma unroll
            for (int q = 0; q < IPL; ++q) {
                const double r[3] = {xi[q] - c0.x, yi[q] - c0.y, zi[q] - c1.x};
                const double r2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
                if (t0 + jj == min(ib + q, bend - 1)) continue;
                if (r2 == 0.0) {
                    bad = 1;
                    continue;
                }
                double o[3];
                oseen_term64(r, F, o);
                for (int c = 0; c < 3; ++c) acc[q][c] = acc[q][c] + o[c];
                if (RPY) {
                    rpy_term64(r, F, o);
                    for (int c = 0; c < 3; ++c) acc[q][3 + c] = acc[q][3 + c] + o[c];
                }
            }
        };
        /* F64_J sources from jj; MASK: some of them may be the group's own
         * targets, whose terms get r2 = 1 and no force */
        auto group = [&](int jj, auto mask_c) {
            constexpr bool MASK = decltype(mask_c)::value;
            double rx[F64_J][IPL], ry[F64_J][IPL], rz[F64_J][IPL], r2[F64_J][IPL];
            Range64 rg;
#pragma unroll
            for (int u = 0; u < F64_J; ++u)
#pragma unroll
                for (int q = 0; q < IPL; ++q) {
                    rx[u][q] = xi[q] - lds.src[0][jj + u].x;
                    ry[u][q] = yi[q] - lds.src[0][jj + u].y;
                    rz[u][q] = zi[q] - lds.src[1][jj + u].x;
                    r2[u][q] = __builtin_fma(rz[u][q], rz[u][q],
                                             __builtin_fma(ry[u][q], ry[u][q], rx[u][q] * rx[u][q]));
                    if (MASK && t0 + jj + u == min(ib + q, bend - 1)) r2[u][q] = 1.0;
                    rg.r2(r2[u][q]);
                }
            if (!__all(rg.ok_r2())) {
                for (int u = 0; u < F64_J; ++u) plain(jj + u);
                return;
            }
#pragma unroll
            for (int u = 0; u < F64_J; ++u) {
                const double Gx = lds.src[1][jj + u].y, Gy = lds.src[2][jj + u].x, Gz = lds.src[2][jj + u].y;
#pragma unroll
                for (int q = 0; q < IPL; ++q) {
                    const bool self = MASK && t0 + jj + u == min(ib + q, bend - 1);
                    const double Fx = self ? 0.0 : Gx, Fy = self ? 0.0 : Gy, Fz = self ? 0.0 : Gz;
                    const double ir = rsqrt64(r2[u][q]), ir2 = ir * ir;
                    const double fr = __builtin_fma(rz[u][q], Fz, __builtin_fma(ry[u][q], Fy, rx[u][q] * Fx));
                    const double tt = fr * ir2;
                    acc[q][0] = __builtin_fma(ir, __builtin_fma(tt, rx[u][q], Fx), acc[q][0]);
                    acc[q][1] = __builtin_fma(ir, __builtin_fma(tt, ry[u][q], Fy), acc[q][1]);
                    acc[q][2] = __builtin_fma(ir, __builtin_fma(tt, rz[u][q], Fz), acc[q][2]);
                    if (RPY) {
                        const double ir3 = ir * ir2, t3 = -3.0 * tt;
                        acc[q][3] = __builtin_fma(ir3, __builtin_fma(t3, rx[u][q], Fx), acc[q][3]);
                        acc[q][4] = __builtin_fma(ir3, __builtin_fma(t3, ry[u][q], Fy), acc[q][4]);
                        acc[q][5] = __builtin_fma(ir3, __builtin_fma(t3, rz[u][q], Fz), acc[q][5]);
                    }
                }
            }
        };
        int jj = 64 * w;
        const int je = jj + n;
        if (t0 + je <= b0 || t0 + jj >= bend)
            for (; jj + F64_J <= je; jj += F64_J) group(jj, std::integral_constant<bool, false>{});
        else
            for (; jj + F64_J <= je; jj += F64_J) group(jj, std::integral_constant<bool, true>{});
        for (; jj < je; ++jj) plain(jj);
    }
    if (bad && ib < bend) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (G > 1) {
        __syncthreads(); /* the last tile is no longer read */
        if (w > 0) {
#pragma unroll
            for (int q = 0; q < IPL; ++q)
#pragma unroll
                for (int c = 0; c < NC; ++c) lds.red[w > 0 ? w - 1 : 0][q * NC + c][l] = acc[q][c];
        }
        __syncthreads();
        if (w > 0) return;
#pragma unroll
        for (int g = 1; g < G; ++g)
#pragma unroll
            for (int q = 0; q < IPL; ++q)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[q][c] = acc[q][c] + lds.red[g - 1][q * NC + c][l];
    }
    const long long base = d.sys_pbase[it.sys] + (long long)it.c * d.ncomp * it.Nb;
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        const int li = ib + q - it.ioff;
        if (ib + q < bend) {
#pragma unroll
            for (int c = 0; c < NC; ++c) d.part[base + (long long)c * it.Nb + li] = acc[q][c];
        }
    }
}

/* Work-group barrier that orders LDS only: vector-memory loads in flight
 * (the step table's next row, the next chunk's sources) are not waited for. */
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

/* AD_FP64 in one kernel, with producer and consumer waves: a work-group owns
 * TW targets of one system. Its NP producer waves form the pair terms of the
 * system's sources in chunks of CW (64 or 128; a lane forms the terms of
 * sources l, l + 64, ... for the TW targets), into LDS rows (component x TW +
 * target) by columns (the chunk's sources); its consumer wave adds them,
 * lane r row r, to a running sum in ascending j. Chunks go in rounds of NP,
 * one per producer, through two sets of buffers: the producers form round
 * m + 1 while the consumer adds round m, and one LDS barrier ends a round.
 * Unless steric forces are on, the consumer, which then holds every sum of
 * its targets, also closes the stage or the product: no partial sums, no
 * second launch (4.7 us per stage at N = 4096).
 * The terms are the plain sum's expressions and the additions its sequence,
 * so the result is bitwise k_pairs_f64's with one chunk per system. The
 * self term, a coincident pair (which raises the flag) and the padding past
 * the system's last source are stored as zeros of either sign and added like
 * the others: a sum that starts at +0.0 is never -0.0 in round-to-nearest, so
 * adding +0.0 or -0.0 changes no bit of it. The consumer's lanes past the last row repeat its
 * reads and additions (the same LDS addresses, served once). */
template <int TW, int NP, int CW, int RPY>
__global__ __launch_bounds__(64 * (NP + 1)) void k_pairs_f64w(Dev d, Epi e, int mode) {
    constexpr int NC = RPY ? 6 : 3;
    constexpr int ROWS = NC * TW;
    constexpr int RS = CW + 2;          /* LDS row stride in doubles: pairs of columns are 16-byte
                                           aligned, and the rows' reads of a pair fall in different
                                           banks (4 mod 64) */
    constexpr int BUF = ROWS * RS; /* doubles per chunk buffer */
    extern __shared__ __align__(16) double w_lds[]; /* [2 sets][NP chunks][ROWS][RS] */
    const Item it = d.fitems[blockIdx.x];
    if (mode && !e.pack_next) advance_slots(d, e);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    const int Nb = it.Nb, off = it.ioff;
    const int nch = (Nb + CW - 1) / CW;
    const int M = (nch + NP - 1) / NP; /* rounds */
    if (w == 0) {
        /* the consumer */
        const int r = l < ROWS ? l : ROWS - 1;
        double acc = 0.0;
        /* inputs of the closing, loaded first: lane a TW + q owns component a
         * of target q, lane q < ni the phase of dumbbell q / 2 */
        const bool close = e.u_aos || e.pack_next;
        const int ca = l / TW, ci = it.i0 + (l - ca * TW);
        const bool cl = l < 3 * TW && l - ca * TW < it.ni;
        double u0 = 0.0, xv = 0.0, rv = 0.0, st = 0.0, ct = 0.0;
        double2 tp = make_double2(0.0, 0.0);
        double nz = 0.0;
        if (close) {
            if (cl) {
                const int o = ca * d.Ntot + ci;
                u0 = d.U0[o];
                if (!e.u_aos) {
                    xv = d.X[o];
                    if (e.stage > 0) rv = d.R[o];
                }
            }
            if (!e.u_aos) {
                const long long step = d.ctl->slot[e.stage > 0];
                advance_step(d, e, step);
                if (cl) nz = stage_noise(e.c, ci, step, ca);
                const long long row = step & (d.ring - 1);
                if (l < it.ni) {
                    st = d.tab[row * 8 + 2 * e.stage];
                    ct = d.tab[row * 8 + 2 * e.stage + 1];
                    tp = d.phitrig[(it.i0 >> 1) + (l >> 1)];
                }
            }
        }
        lds_barrier();
        for (int m = 0; m < M; ++m) {
            const double* S = w_lds + (m & 1) * NP * BUF + r * RS;
            for (int p = 0; p < NP && m * NP + p < nch; ++p) {
                /* two columns per read, a batch of reads ahead of the
                 * additions (9.6 cycles per column against 16.1 one column
                 * at a time; the dependent additions alone take 7.3) */
                const double2* Ta = reinterpret_cast<const double2*>(S + p * BUF);
                constexpr int B = 8;
                double2 v[B];
#pragma unroll
                for (int u = 0; u < B; ++u) v[u] = Ta[u];
#pragma unroll
                for (int c = 0; c < CW / 2; c += B) {
                    double2 nx[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) nx[u] = (c + B < CW / 2) ? Ta[c + B + u] : v[u];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        acc = acc + v[u].x;
                        acc = acc + v[u].y;
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) v[u] = nx[u];
                }
            }
            lds_barrier();
        }
        if (!close) {
            /* steric forces on: the epilogue and the steric kernel close */
            if (l < ROWS) {
                const int a = l / TW, q = l - a * TW;
                if (q < it.ni) d.part[d.sys_pbase[it.sys] + (long long)a * Nb + (it.i0 + q - off)] = acc;
            }
            return;
        }
        /* The consumer holds every sum of its targets: it closes the stage
         * (or the product) as the epilogue does, in the epilogue's order. */
        const double corr = RPY ? __shfl(acc, (l + 3 * TW) & 63) : 0.0;
        double y = 0.0;
        int nf = 0;
        if (cl) {
            double k = u0 + e.c.co * acc;
            if (RPY) k = k + e.c.cr * corr;
            nf = !isfinite(k);
            if (e.u_aos)
                e.u_aos[3 * ci + ca] = k;
            else
                y = stage_update(d, e, ca * d.Ntot + ci, k, xv, rv, nz);
        }
        if (__any(nf) && l == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
        if (e.u_aos) return;
        /* lane q < TW: sphere q; both lanes of a dumbbell evaluate the same
         * forces */
        const int pq = l & (TW - 1), q0 = pq & ~1;
        double y0[3], y1[3], f0[3], f1[3];
        for (int a = 0; a < 3; ++a) {
            y0[a] = __shfl(y, a * TW + q0);
            y1[a] = __shfl(y, a * TW + q0 + 1);
        }
        if (l < it.ni) {
            spring_forces(e.c, y0, y1, tp.x, tp.y, st, ct, f0, f1);
            const int i = it.i0 + l;
            const bool up = l & 1;
            double ys[3], fs[3];
            for (int a = 0; a < 3; ++a) {
                ys[a] = up ? y1[a] : y0[a];
                fs[a] = up ? f1[a] : f0[a];
                d.U0[a * d.Ntot + i] = e.c.cs * fs[a];
            }
            d.pD2[3 * i + 0] = make_double2(ys[0], ys[1]);
            d.pD2[3 * i + 1] = make_double2(ys[2], fs[0]);
            d.pD2[3 * i + 2] = make_double2(fs[1], fs[2]);
        }
        return;
    }
    /* producer p forms chunk m NP + p of every round m */
    const int p = w - 1;
    double xi[TW], yi[TW], zi[TW];
    int iq[TW];
    bool okq[TW];
#pragma unroll
    for (int q = 0; q < TW; ++q) {
        okq[q] = q < it.ni;
        iq[q] = it.i0 + (okq[q] ? q : 0);
        const double2 p0 = d.pD[3 * iq[q]], p1 = d.pD[3 * iq[q] + 1];
        xi[q] = p0.x; yi[q] = p0.y; zi[q] = p1.x;
    }
    int bad = 0;
    constexpr int U = CW / 64; /* sources per lane and chunk */
    double2 s0[U], s1[U], s2[U]; /* the sources of the next chunk to form */
    auto load = [&](int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int lj = k * CW + u * 64 + l;
            const int j = off + (lj < Nb ? lj : Nb - 1);
            s0[u] = d.pD[3 * j];
            s1[u] = d.pD[3 * j + 1];
            s2[u] = d.pD[3 * j + 2];
        }
    };
    /* The terms of chunk k by the plain expressions, for any operands. */
    auto form_plain = [&](int k, double* Tb0) {
#pragma unroll 1
        for (int u = 0; u < U; ++u) {
            const int lj = k * CW + u * 64 + l;
            const bool in = lj < Nb;
            double* Tb = Tb0 + u * 64 + l;
            const double xj = u ? s0[U - 1].x : s0[0].x, yj = u ? s0[U - 1].y : s0[0].y;
            const double zj = u ? s1[U - 1].x : s1[0].x, Fx = u ? s1[U - 1].y : s1[0].y;
            const double Fy = u ? s2[U - 1].x : s2[0].x, Fz = u ? s2[U - 1].y : s2[0].y;
#pragma unroll
            for (int q = 0; q < TW; ++q) {
                const double r[3] = {xi[q] - xj, yi[q] - yj, zi[q] - zj};
                const double F[3] = {Fx, Fy, Fz};
                const double r2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
                const bool self = off + lj == iq[q];
                double t[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
                if (in && !self && r2 != 0.0) {
                    oseen_term64(r, F, t);
                    if (RPY) rpy_term64(r, F, v);
                }
                bad |= in && okq[q] && !self && r2 == 0.0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    Tb[(a * TW + q) * RS] = t[a];
                    if (RPY) Tb[((3 + a) * TW + q) * RS] = v[a];
                }
            }
        }
    };
    /* The same terms by the shared short forms (rcp_sqrt_exact and the
     * following), or form_plain where some lane's operands lie outside their
     * range. MASK: the chunk holds one of the targets or ends past the
     * system's last source; those terms get ir = 0, so they are +-0.0, and a
     * sum that started at +0.0 does not change when either is added. */
    auto form_any = [&](int k, double* Tb0, auto mask_c) {
        constexpr bool MASK = decltype(mask_c)::value;
        double rx[U][TW], ry[U][TW], rz[U][TW], r2[U][TW], fr[U][TW], ir[U][TW], iy[U][TW];
        bool skip[U][TW];
        Range64 rg;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int lj = k * CW + u * 64 + l;
            const double Fx = s1[u].y, Fy = s2[u].x, Fz = s2[u].y;
#pragma unroll
            for (int q = 0; q < TW; ++q) {
                rx[u][q] = xi[q] - s0[u].x;
                ry[u][q] = yi[q] - s0[u].y;
                rz[u][q] = zi[q] - s1[u].x;
                r2[u][q] = (rx[u][q] * rx[u][q] + ry[u][q] * ry[u][q]) + rz[u][q] * rz[u][q];
                if (MASK) {
                    skip[u][q] = lj >= Nb || off + lj == iq[q];
                    r2[u][q] = skip[u][q] ? 1.0 : r2[u][q];
                }
                fr[u][q] = (rx[u][q] * Fx + ry[u][q] * Fy) + rz[u][q] * Fz;
                rg.r2(r2[u][q]);
                rg.fr(fr[u][q]);
                double s;
                rcp_sqrt_exact(r2[u][q], s, ir[u][q], iy[u][q], rg.ones);
            }
        }
        bool ok = rg.ok();
        if (__any(rg.small_fr())) { /* zero forces, as a rule */
            asm volatile("" ::: "memory"); /* keeps the tests from being hoisted */
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < TW; ++q) ok = ok && Range64::fr_fits(fr[u][q]);
        }
        if (__any(!ok)) {
            form_plain(k, Tb0);
            return;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double* Tb = Tb0 + u * 64 + l;
            const double Fx = s1[u].y, Fy = s2[u].x, Fz = s2[u].y;
#pragma unroll
            for (int q = 0; q < TW; ++q) {
                const double tt = div_exact(fr[u][q], r2[u][q], iy[u][q]);
                const double iv = MASK && skip[u][q] ? 0.0 : ir[u][q];
                Tb[(0 * TW + q) * RS] = iv * (Fx + tt * rx[u][q]);
                Tb[(1 * TW + q) * RS] = iv * (Fy + tt * ry[u][q]);
                Tb[(2 * TW + q) * RS] = iv * (Fz + tt * rz[u][q]);
                if (RPY) {
                    const double ir3 = div_exact(iv, r2[u][q], iy[u][q]);
                    const double t3 = 3.0 * tt;
                    Tb[(3 * TW + q) * RS] = ir3 * (Fx - t3 * rx[u][q]);
                    Tb[(4 * TW + q) * RS] = ir3 * (Fy - t3 * ry[u][q]);
                    Tb[(5 * TW + q) * RS] = ir3 * (Fz - t3 * rz[u][q]);
                }
            }
        }
    };
    const int own = it.i0 - off; /* local index of the first target */
    auto form = [&](int k, double* Tb0) {
        if ((k * CW < own + TW && (k + 1) * CW > own) || (k + 1) * CW > Nb)
            form_any(k, Tb0, std::integral_constant<bool, true>{});
        else
            form_any(k, Tb0, std::integral_constant<bool, false>{});
    };
    load(p);
    form(p, w_lds + p * BUF);
    load(NP + p);
    lds_barrier();
    for (int m = 0; m < M; ++m) {
        if (m + 1 < M) {
            form((m + 1) * NP + p, w_lds + (((m + 1) & 1) * NP + p) * BUF);
            load((m + 2) * NP + p);
        }
        lds_barrier();
    }
    if (__any(bad) && l == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
}

/* Steric sum of sphere i over its candidate list (FP32C path). The list holds
 * every source that was closer than rc + skin at the previous stage; it is
 * sorted so that the terms are added in ascending j, exactly as the full
 * sum would add them, and then emptied for the next pair sum. */
__device__ int steric_list(const Dev& d, const Coef& c, int i, double acc[3], int* any) {
    const int N = d.Ntot;
    int n = d.nbr_cnt[i];
    n = n < NBR_CAP ? n : NBR_CAP; /* an overflow was flagged when it happened */
    n = n > 0 ? n : 0;
    int idx[NBR_CAP];
    for (int k = 0; k < n; ++k) {
        const int j = d.nbr_idx[i * NBR_CAP + k];
        idx[k] = (j >= 0 && j < N) ? j : i; /* entries come from the pair kernel; i itself is skipped */
    }
    for (int k = 1; k < n; ++k) { /* insertion sort, n <= NBR_CAP */
        const int v = idx[k];
        int m = k - 1;
        while (m >= 0 && idx[m] > v) {
            idx[m + 1] = idx[m];
            --m;
        }
        idx[m + 1] = v;
    }
    const double xi[3] = {d.Y[i], d.Y[N + i], d.Y[2 * N + i]};
    const double rc2 = c.rc * c.rc;
    int bad = 0;
    acc[0] = acc[1] = acc[2] = 0.0;
    *any = 0;
    for (int k = 0; k < n; ++k) {
        const int j = idx[k];
        if (j == i) continue;
        const double rx = xi[0] - d.Y[j], ry = xi[1] - d.Y[N + j], rz = xi[2] - d.Y[2 * N + j];
        const double r2 = (rx * rx + ry * ry) + rz * rz;
        if (r2 >= rc2) continue;
        if (r2 == 0.0) {
            bad = 1;
            continue;
        }
        const double r = sqrt(r2);
        const double cc = c.ks * (c.rc - r) / r;
        acc[0] = acc[0] + cc * rx;
        acc[1] = acc[1] + cc * ry;
        acc[2] = acc[2] + cc * rz;
        *any = 1;
    }
    d.nbr_cnt[i] = 0;
    return bad;
}

/* steric forces at the stage positions Y, then the pack: from the candidate
 * lists when the pair kernel records them (LIST), else by the full sum */
template <int LIST, int IT>
__global__ __launch_bounds__(256) void k_steric_pack(Dev d, Coef c, int prec) {
    int s0;
    const int s = steric_dumbbell<IT>(d, s0);
    if (IT == 0 && s < 0) return;
    const int N = d.Ntot;
    const int i0 = 2 * max(s, 0);
    double y0[3], y1[3], f0[3], f1[3];
    for (int a = 0; a < 3; ++a) {
        y0[a] = d.Y[a * N + i0];
        y1[a] = d.Y[a * N + i0 + 1];
        f0[a] = d.Fs[a * N + i0];
        f1[a] = d.Fs[a * N + i0 + 1];
    }
    int bad = 0;
    if (LIST) {
        double acc[3];
        int any;
        bad |= steric_list(d, c, i0, acc, &any);
        if (any)
            for (int a = 0; a < 3; ++a) f0[a] = f0[a] + acc[a];
        bad |= steric_list(d, c, i0 + 1, acc, &any);
        if (any)
            for (int a = 0; a < 3; ++a) f1[a] = f1[a] + acc[a];
    } else {
        auto get = [&](int j, double x[3]) {
            x[0] = d.Y[j];
            x[1] = d.Y[N + j];
            x[2] = d.Y[2 * N + j];
        };
        bad |= add_steric<IT>(d, c, s, s0, get, f0, f1);
    }
    if (bad) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
    if (s < 0) return;
    store_pack(d, c, prec, i0, y0, y1, f0, f1, 1);
}

/* Records: dumbbell centres and per-system mean position. The mean is the sum
 * in ascending j divided by the count, as the oracle forms it, so its
 * additions are one dependent chain per (system, component): what bounds the
 * kernel is that chain's latency, one FP64 addition after another. The first
 * nsys work-groups take one system each: three waves (one per component) copy
 * tiles of REC_T spheres into LDS, double buffered, while lanes 0 to 2 of the
 * first wave add the tile before in order, their LDS reads a batch ahead of
 * the additions. The remaining work-groups write the centres. (One thread per
 * component reading global memory ran at the load latency: 306 us per record
 * at 4096 spheres and 5027 us at 65536, against 24 and 353; 142
 * us for 512 systems of up to 800 spheres, against 9.) BY_THREADS is that form,
 * for ensembles whose systems are many and small: a work-group costs about 1 ns
 * of the chip, an addition from memory 0.07 us of its thread, so it is taken
 * from 64 systems per sphere of the largest one (us per record, work-groups
 * and threads: 30000 dumbbells 29 and 2, 8192 systems of 16 spheres 11.0 and
 * 5.4, 4096 6.5 and 4.3; 1024 of 54 3.5 and 11.4). */
constexpr int REC_WG = 256;
constexpr int REC_T = 512;  /* spheres per tile */
constexpr int REC_RS = REC_T + 2; /* LDS row stride: even, so that pairs are 16-byte aligned */
constexpr int REC_U = 16;   /* additions per batch of LDS reads */

template <int BY_THREADS>
__global__ __launch_bounds__(REC_WG) void k_record(Dev d, double* __restrict__ centres, double* __restrict__ com,
                                                   int ncom) {
    __shared__ __align__(16) double tile[2][3][BY_THREADS ? 2 : REC_RS];
    const int N = d.Ntot;
    if ((int)blockIdx.x >= ncom) {
        const int g = (blockIdx.x - ncom) * REC_WG + threadIdx.x;
        if (centres && g < d.Stot)
            for (int a = 0; a < 3; ++a)
                centres[3 * g + a] = 0.5 * (d.X[a * N + 2 * g] + d.X[a * N + 2 * g + 1]);
        return;
    }
    if constexpr (BY_THREADS) {
        const int g = blockIdx.x * REC_WG + threadIdx.x;
        if (g < 3 * d.nsys) {
            const int b = g / 3, a = g % 3;
            const int j0 = d.sys_off[b], j1 = d.sys_off[b + 1];
            double sum = 0.0;
            for (int j = j0; j < j1; ++j) sum = sum + d.X[a * N + j];
            com[3 * b + a] = sum / (double)(j1 - j0);
        }
        return;
    }
    const int b = blockIdx.x;
    const int j0 = d.sys_off[b], n = d.sys_off[b + 1] - j0;
    const int nt = (n + REC_T - 1) / REC_T;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    auto fill = [&](int k) {
        if (w == 0) return;
        const double* x = d.X + (size_t)(w - 1) * N + j0 + k * REC_T;
        double* row = tile[k & 1][w - 1];
        const int m = min(REC_T, n - k * REC_T);
        double v[REC_T / 64];
#pragma unroll
        for (int u = 0; u < REC_T / 64; ++u) v[u] = (u * 64 + l < m) ? x[u * 64 + l] : 0.0;
#pragma unroll
        for (int u = 0; u < REC_T / 64; ++u) row[u * 64 + l] = v[u];
    };
    double sum = 0.0;
    fill(0);
    __syncthreads();
    for (int k = 0; k < nt; ++k) {
        if (k + 1 < nt) fill(k + 1);
        if (w == 0 && l < 3) {
            const double* row = tile[k & 1][l];
            const int m = min(REC_T, n - k * REC_T);
            const int mb = m / REC_U;
            double v[REC_U], q[REC_U];
            if (mb > 0) {
#pragma unroll
                for (int u = 0; u < REC_U; ++u) v[u] = row[u];
            }
            for (int c = 0; c < mb; ++c) {
                /* the next batch (at most 2 past the row's end: its padding) */
                const double* nx = row + min((c + 1) * REC_U, REC_RS - REC_U);
#pragma unroll
                for (int u = 0; u < REC_U; ++u) q[u] = nx[u];
#pragma unroll
                for (int u = 0; u < REC_U; ++u) sum = sum + v[u];
#pragma unroll
                for (int u = 0; u < REC_U; ++u) v[u] = q[u];
            }
            for (int u = mb * REC_U; u < m; ++u) sum = sum + row[u];
        }
        __syncthreads();
    }
    if (w == 0 && l < 3) com[3 * b + l] = sum / (double)n;
}

/* ------------------------------------------------------- resident small systems */

/* Stage update of one component, in the operation order of stage_update,
 * with the RK accumulator r and the state x held by the caller. */
__device__ __forceinline__ double res_update(const Coef& c, int integ, int stage, int nst, double k, double& x,
                                             double& r, double nz) {
    double y;
    if (integ == 0) {
        if (stage == 0) {
            r = k;
            y = x + c.h2 * k;
        } else if (stage == 1) {
            r = r + 2.0 * k;
            y = x + c.h2 * k;
        } else if (stage == 2) {
            r = r + 2.0 * k;
            y = x + c.dt * k;
        } else {
            y = x + c.dt6 * (r + k);
        }
    } else {
        if (stage == 0) {
            r = k;
            y = x + c.dt * k;
        } else {
            y = x + c.h2 * (r + k);
        }
        if (c.noise) y = y + nz;
    }
    if (stage == nst - 1) x = y;
    return y;
}

/* Resident form (ad_launch.fused = 4): one work-group per system holds the
 * system on chip and runs every stage of nsteps steps in one launch, with
 * work-group barriers between the phases of a stage. The state comes from
 * and returns to d.X; the first stage's forces are formed at
 * (st0, ct0) = (sin, cos)(omega t) of step step0, and every later stage's
 * at the step table's row, the next step's row loaded while a step runs. */

/* One level of the fixed butterfly that combines the (hi, lo) sums
 * v = (hi.x, lo.x, hi.y, lo.y, hi.z, lo.z) of adjacent lanes: each lane takes
 * the sums of lane (itself xor distance) and adds them in with TwoSum. */
__device__ __forceinline__ void combine_hilo(float v[6], const float o[6]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) add_hilo(v[2 * a], v[2 * a + 1], o[2 * a], o[2 * a + 1]);
}
/* distances 1 and 2 through DPP quad permutations (CTRL 0xB1 swaps the lanes
 * of each pair, 0x4E the pairs of each quad): a VALU operation, no LDS round
 * trip */
template <int CTRL>
__device__ __forceinline__ void combine_level_dpp(float v[6]) {
    float o[6];
#pragma unroll
    for (int q = 0; q < 6; ++q)
        o[q] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v[q]), CTRL, 0xF,
                                                                     0xF, false));
    combine_hilo(v, o);
}
/* larger distances (uniform over the wave) through ds_bpermute */
__device__ __forceinline__ void combine_level_shfl(float v[6], int sh) {
    float o[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) o[q] = __shfl_xor(v[q], sh);
    combine_hilo(v, o);
}

/* FP64 (the plain sum, bitwise that of the sequential oracle): X, R, Y, F
 * and the pair sums in LDS. Per stage: the terms of a chunk of source
 * columns are evaluated in parallel into an LDS matrix, then every
 * (target, component) thread adds its row of the chunk in ascending j and
 * closes it (velocity, stage update, next stage position); then one thread
 * per sphere forms the next stage's spring force (both threads of a dumbbell
 * evaluate them from the same inputs, so they agree bit for bit).
 * What bounds it is the length of that chain, of which four barriers, two
 * square roots and three divisions in a row were the larger part. Up to 16
 * spheres no thread has more than one pair: it forms its source's spring force
 * itself, next to the pair's separation, so both square roots and the
 * reciprocals run side by side (rcp_sqrt_exact), and a stage has two barriers.
 * With more, a thread has several pairs one after another and would form a
 * spring force for each, so they keep the springs' own phase. RK4 step, before
 * and after: 2 spheres 4.04 and 3.88 us, 6 4.62 and 3.76, 14
 * 4.95 and 4.15, 16 4.35 and 3.80 (RPY 5.10 and 4.48); Heun with noise, 16
 * spheres: 3.92 and 2.44 us (the noise, the same in both stages, is formed in
 * the first).
 * ONE = 0 is the kernel without that form, for more systems than are resident
 * at once with it: 84 registers in place of 103, see resident_forms. */
template <int RPY, int INTEG, int ONE>
__global__ __launch_bounds__(RES_T, !ONE && RPY && INTEG == 2 ? 4 : 1) void k_resident(Dev d, Epi e, long long step0, int nsteps, double st0,
                                                    double ct0) {
    /* INTEG: 0 RK4, 1 Heun, 2 Heun with noise; the stages are unrolled, so
     * every stage's update and table entries are fixed at compile time */
    constexpr int NST = INTEG == 0 ? 4 : 2;
    constexpr int T = RES_T;
    extern __shared__ double res_lds[];
    const Item it = d.fitems[blockIdx.x];
    const int n = it.Nb, ioff = it.ioff;
    const int N = d.Ntot;
    const int tid = threadIdx.x;
    const Coef& c = e.c;
    double* X = res_lds;
    double* R = X + 3 * n;
    double* Y = R + 3 * n;
    double* F = Y + 3 * n;
    double* Acc = F + 3 * n; /* pair sums [3][n] (RPY: then [3][n]) */
    double* Bcc = Acc + 3 * n;
    double* Tm = reinterpret_cast<double*>(reinterpret_cast<char*>(res_lds) +
                                           ((3 * n * (5 + (RPY ? 1 : 0))) * 8 + 15) / 16 * 16);
    const int cc = resident_cols(n, RPY);
    /* the chunk's terms [3][n][cs]: a row of cs (odd) doubles, so that the
     * threads of consecutive targets read distinct LDS banks */
    const int cs = resident_col_stride(cc);
    double* Tb = Tm + 3 * n * cs; /* RPY corrections of the chunk */

    for (int q = tid; q < 3 * n; q += T) {
        const int a = q / n, i = q - a * n;
        const double v = d.X[a * N + ioff + i];
        X[q] = v;
        Y[q] = v;
    }
    /* one: at most one pair per thread, (pi, pj), which forms sphere pj's
     * spring force itself; else thread tid < n forms sphere tid's */
    const bool one = ONE && n * n <= T;
    const int pi = one ? tid / n : 0, pj = one ? tid - pi * n : tid;
    const bool springs = tid < (one ? n * n : n);
    double2 tp = make_double2(0.0, 0.0);
    if (springs) tp = d.phitrig[(ioff >> 1) + (pj >> 1)];
    int bad = 0;
    /* the step table's row index in a vector register: its loads are then
     * vector loads, which the LDS-only barriers do not wait for */
    int row = (int)(step0 & (d.ring - 1));
    asm volatile("" : "+v"(row));
    double tb[8], nb[8];
    for (int q = 0; q < 8; ++q) tb[q] = nb[q] = 0.0;
    if (springs)
        for (int q = 0; q < 8; ++q) tb[q] = d.tab[row * 8 + q];
    __syncthreads();

    auto forces = [&](double st, double ct) {
        if (tid < n) {
            const int i0 = tid & ~1;
            double y0[3], y1[3], f0[3], f1[3];
            for (int a = 0; a < 3; ++a) {
                y0[a] = Y[a * n + i0];
                y1[a] = Y[a * n + i0 + 1];
            }
            spring_forces(c, y0, y1, tp.x, tp.y, st, ct, f0, f1);
            for (int a = 0; a < 3; ++a) F[a * n + tid] = (tid & 1) ? f1[a] : f0[a];
        }
        lds_barrier();
    };
    auto store_term = [&](int o, const double t[3], const double tq[3]) {
        const int m = n * cs; /* component stride */
        for (int a = 0; a < 3; ++a) {
            Tm[a * m + o] = t[a];
            if (RPY) Tb[a * m + o] = tq[a];
        }
    };
    /* the spring force of sphere pj, kept by its own pair's thread, and the
     * term of the pair (pi, pj), their square roots and divisions together by
     * the short forms where those hold */
    auto pair_of_one = [&](double st, double ct) {
        const int i0 = pj & ~1;
        double y0[3], y1[3], r[3], Fj[3], F0[3], t[3] = {0.0, 0.0, 0.0}, tq[3] = {0.0, 0.0, 0.0};
        for (int a = 0; a < 3; ++a) {
            y0[a] = Y[a * n + i0];
            y1[a] = Y[a * n + i0 + 1];
            r[a] = Y[a * n + pi] - ((pj & 1) ? y1[a] : y0[a]);
        }
        const double nv[3] = {y1[0] - y0[0], y1[1] - y0[1], y1[2] - y0[2]};
        const double n2 = (nv[0] * nv[0] + nv[1] * nv[1]) + nv[2] * nv[2];
        const bool self = pi == pj;
        const double r2 = self ? 1.0 : (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
        Range64 rg;
        double dd, id, iy, rr, ir, iz;
        rcp_sqrt_exact(n2, dd, id, iy, rg.ones);
        rcp_sqrt_exact(r2, rr, ir, iz, rg.ones);
        const double pull = -c.k * (dd - (c.ell + c.lam * (st * tp.y + ct * tp.x)));
        const double cc1 = div_exact(pull, dd, id);
        for (int a = 0; a < 3; ++a) Fj[a] = (pj & 1) ? cc1 * nv[a] : -(cc1 * nv[a]);
        const double fr = (r[0] * Fj[0] + r[1] * Fj[1]) + r[2] * Fj[2];
        rg.r2(n2);
        rg.r2(r2);
        rg.fr(pull);
        rg.fr(fr);
        if (__builtin_expect(rg.ok() && (!rg.small_fr() || (Range64::fr_fits(pull) && Range64::fr_fits(fr))), 1)) {
            const double tt = div_exact(fr, r2, iz);
            for (int a = 0; a < 3; ++a) t[a] = ir * (Fj[a] + tt * r[a]);
            if (RPY) {
                const double ir3 = div_exact(ir, r2, iz), t3 = 3.0 * tt;
                for (int a = 0; a < 3; ++a) tq[a] = ir3 * (Fj[a] - t3 * r[a]);
            }
        } else {
            double f1[3];
            spring_forces(c, y0, y1, tp.x, tp.y, st, ct, F0, f1);
            for (int a = 0; a < 3; ++a) Fj[a] = (pj & 1) ? f1[a] : F0[a];
            if (r2 != 0.0) {
                oseen_term64(r, Fj, t);
                if (RPY) rpy_term64(r, Fj, tq);
            } else {
                bad = 1;
            }
        }
        if (self) {
            for (int a = 0; a < 3; ++a) {
                F[a * n + pj] = Fj[a];
                t[a] = tq[a] = 0.0;
            }
        }
        store_term(pi * cs + pj, t, tq);
    };
    double noise[2] = {0.0, 0.0}; /* of this thread's at most two rows */
    static_assert(3 * RES_MAX64 <= 2 * RES_T, "rows per thread");
    double fst = st0, fct = ct0; /* the time of the next forces */
    if (!one) forces(fst, fct);

    auto stage_pass = [&](auto one_c, auto stage_c, long long step) {
        constexpr bool one = decltype(one_c)::value;
        constexpr int stage = decltype(stage_c)::value;
        for (int j0 = 0; j0 < n; j0 += cc) {
            const int nc = min(cc, n - j0);
            if constexpr (one) {
                if (springs) pair_of_one(fst, fct);
            } else {
                for (int p = tid; p < n * nc; p += T) {
                    const int i = p / nc, jj = p - i * nc, j = j0 + jj;
                    const double r[3] = {Y[i] - Y[j], Y[n + i] - Y[n + j], Y[2 * n + i] - Y[2 * n + j]};
                    const double r2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
                    double t[3] = {0.0, 0.0, 0.0}, tq[3] = {0.0, 0.0, 0.0};
                    if (j != i && r2 != 0.0) {
                        const double Fj[3] = {F[j], F[n + j], F[2 * n + j]};
                        oseen_term64(r, Fj, t);
                        if (RPY) rpy_term64(r, Fj, tq);
                    } else if (j != i) {
                        bad = 1;
                    }
                    store_term(i * cs + jj, t, tq);
                }
            }
            lds_barrier();
            /* one thread per (component, target): the target's row of the
             * chunk in ascending j, its LDS loads eight at a time */
            for (int q = tid; q < 3 * n; q += T) {
                const double* row = Tm + q * cs; /* component q / n of target q mod n */
                const double* rowb = Tb + q * cs;
                /* The self term was stored as a zero and is added like the
                 * others: a sum that starts at +0.0 is never -0.0 in
                 * round-to-nearest, so adding a zero leaves it unchanged, bit
                 * for bit the sum that skips j = i. */
                double acc = (j0 == 0) ? 0.0 : Acc[q];
                double bcc = (RPY && j0 > 0) ? Bcc[q] : 0.0;
                int jb = 0;
                for (; jb + 8 <= nc; jb += 8) {
                    double v[8], w[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        v[u] = row[jb + u];
                        w[u] = RPY ? rowb[jb + u] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        acc = acc + v[u];
                        if (RPY) bcc = bcc + w[u];
                    }
                }
                if constexpr (one) { /* the rest together too, +0.0 past the end */
                    double v[8], w[8];
                    if (jb < nc) {
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const int at = min(jb + u, nc - 1);
                            v[u] = row[at];
                            w[u] = RPY ? rowb[at] : 0.0;
                        }
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            acc = acc + (jb + u < nc ? v[u] : 0.0);
                            if (RPY) bcc = bcc + (jb + u < nc ? w[u] : 0.0);
                        }
                    }
                } else {
                    for (; jb < nc; ++jb) {
                        acc = acc + row[jb];
                        if (RPY) bcc = bcc + rowb[jb];
                    }
                }
                Acc[q] = acc;
                if (RPY) Bcc[q] = bcc;
            }
            if (!one && j0 + cc < n) lds_barrier(); /* before the next chunk's terms */
        }
        /* closing: each thread the (component, sphere) rows that it summed */
        for (int q = tid, w = 0; q < 3 * n; q += T, ++w) {
            const int a = (q >= n) + (q >= 2 * n), i = q - a * n, o = q;
            double k = c.cs * F[o] + c.co * Acc[o];
            if (RPY) k = k + c.cr * Bcc[o];
            if (!isfinite(k)) bad = 1;
            double nz = 0.0;
            if (INTEG == 2) { /* a step's two stages add the same noise */
                if (stage == 0) {
                    nz = c.g * gauss_component(c.seed, ioff + i, step, a);
                    noise[w ? 1 : 0] = nz;
                } else {
                    nz = w ? noise[1] : noise[0];
                }
            }
            double x = X[o], r = R[o];
            Y[o] = res_update(c, INTEG == 0 ? 0 : 1, stage, NST, k, x, r, nz);
            X[o] = x;
            R[o] = r;
        }
        lds_barrier();
        fst = tb[2 * stage];
        fct = tb[2 * stage + 1];
        if (!one) forces(fst, fct);
    };
    auto run = [&](auto one_c) {
        for (int sn = 0; sn < nsteps; ++sn) {
            const long long step = step0 + sn;
            row = row + 1 == d.ring ? 0 : row + 1;
            if (springs)
                for (int q = 0; q < 8; ++q) nb[q] = d.tab[row * 8 + q];
            stage_pass(one_c, std::integral_constant<int, 0>{}, step);
            stage_pass(one_c, std::integral_constant<int, 1>{}, step);
            if constexpr (NST == 4) {
                stage_pass(one_c, std::integral_constant<int, 2>{}, step);
                stage_pass(one_c, std::integral_constant<int, 3>{}, step);
            }
            for (int q = 0; q < 8; ++q) tb[q] = nb[q];
        }
    };
    if constexpr (ONE) {
        if (one) run(std::integral_constant<bool, true>{});
    }
    if (!one) run(std::integral_constant<bool, false>{});
    for (int q = tid; q < 3 * n; q += T) {
        const int a = q / n, i = q - a * n;
        d.X[a * N + ioff + i] = X[q];
    }
    if (__syncthreads_or(bad) && tid == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
}

/* FP32C: the state in registers, only the float pack in LDS. Target sphere
 * t of the system has `split` adjacent lanes (a power of two <= 32, so a
 * dumbbell's lanes lie in one wave); lane 0 of them, the sphere's own lane,
 * holds its FP64 state x, RK accumulator r, stage position y and
 * self-and-partner velocity u0. Per stage:
 *   pair sums: each of the split lanes takes every split-th source in
 *   ascending order (own dumbbell masked by a zero 1/r), folding into
 *   (hi, lo) with TwoSum every 32 sources; the lanes are combined in a
 *   fixed butterfly;
 *   closing in the own lane: velocity, stage update, next stage position;
 *   next forces in the own lane: the partner's position by a lane exchange,
 *   the spring forces (both lanes of a dumbbell evaluate the same
 *   expression), u0 (the partner term reusing the spring's 1/d), and the
 *   sphere's pack entry, written into the other of two pack buffers;
 * then one work-group barrier. Stage s reads buffer s mod 2 and writes the
 * other, and every read of a buffer precedes the barrier that precedes its
 * next write. */
template <int SPLIT, int RPY, int T, int INTEG>
__global__ __launch_bounds__(T) void k_resident_c(Dev d, Epi e, long long step0, int nsteps, double st0,
                                                  double ct0) {
    /* INTEG: 0 RK4, 1 Heun, 2 Heun with noise; the stages are unrolled, so
     * every stage's update and table entries are fixed at compile time */
    constexpr int NST = INTEG == 0 ? 4 : 2;
    extern __shared__ float4 rc_lds[];
    const Item it = d.fitems[blockIdx.x];
    const int n = it.Nb, ioff = it.ioff;
    const int N = d.Ntot;
    const int tid = threadIdx.x;
    const Coef& c = e.c;
    const int split = resident_split(n, T);
    const int t = tid >> __builtin_ctz(split), sub = tid & (split - 1);
    const bool own = t < n && sub == 0;
    const int h = t & 1;
    const int pstride = resident_pack_f4(n); /* float4 per pack buffer */

    double x[3], r[3], y[3], u0[3];
    double2 tp = make_double2(0.0, 0.0);
    double tb[8], nb[8];
    for (int a = 0; a < 3; ++a) x[a] = r[a] = y[a] = u0[a] = 0.0;
    for (int q = 0; q < 8; ++q) tb[q] = nb[q] = 0.0;
    /* the step table's row index, held in a vector register so that its
     * loads are vector loads, which the LDS waits and barriers do not wait
     * for (a scalar load would be waited for by every LDS wait) */
    int row = (int)(step0 & (d.ring - 1));
    asm volatile("" : "+v"(row));
    if (own) {
        for (int a = 0; a < 3; ++a) x[a] = y[a] = d.X[a * N + ioff + t];
        tp = d.phitrig[(ioff >> 1) + (t >> 1)];
        for (int q = 0; q < 8; ++q) tb[q] = d.tab[row * 8 + q];
    }
    int bad = 0;

    auto forces = [&](double st, double ct, int buf) {
        double yp[3];
        for (int a = 0; a < 3; ++a) yp[a] = __shfl_xor(y[a], split);
        if (own) {
            /* lower and upper sphere of the dumbbell, by value selects (a
             * select of array pointers would put the arrays in scratch) */
            double ya[3], yb[3], f0[3], f1[3], f[3], fp[3];
            for (int a = 0; a < 3; ++a) {
                ya[a] = h ? yp[a] : y[a];
                yb[a] = h ? y[a] : yp[a];
            }
            const double id = spring_forces_rs(c, ya, yb, tp.x, tp.y, st, ct, f0, f1);
            for (int a = 0; a < 3; ++a) {
                f[a] = h ? f1[a] : f0[a];
                fp[a] = h ? f0[a] : f1[a];
            }
            /* r = y - yp is +-(y1 - y0) exactly, so 1/|r| is the spring's 1/d */
            const double rr[3] = {y[0] - yp[0], y[1] - yp[1], y[2] - yp[2]};
            const double ir2 = id * id;
            const double tt = ((rr[0] * fp[0] + rr[1] * fp[1]) + rr[2] * fp[2]) * ir2;
            for (int a = 0; a < 3; ++a) {
                double u = c.cs * f[a] + c.co * (id * (fp[a] + tt * rr[a]));
                if (RPY) u = u + c.cr * ((id * ir2) * (fp[a] - (3.0 * tt) * rr[a]));
                u0[a] = u;
            }
            float hi[3], lo[3];
            for (int a = 0; a < 3; ++a) split_f32(y[a], hi[a], lo[a]);
            float4* pA = rc_lds + buf * pstride;
            float4* pB = pA + n;
            float* pz = reinterpret_cast<float*>(pB + n);
            pA[t] = make_float4(hi[0], hi[1], hi[2], (float)f[0]);
            pB[t] = make_float4(lo[0], lo[1], lo[2], (float)f[1]);
            pz[t] = (float)f[2];
        }
        lds_barrier();
    };

    int buf = 0;
    forces(st0, ct0, buf);
    const float crr = c.crr;
    auto stage_pass = [&](auto stage_c, long long step) {
        constexpr int stage = decltype(stage_c)::value;
        const float4* pA = rc_lds + buf * pstride;
        const float4* pB = pA + n;
        const float* pz = reinterpret_cast<const float*>(pB + n);
        float ax = 0.f, ay = 0.f, az = 0.f, bx = 0.f, by = 0.f, bz = 0.f;
        if (t < n) {
            const float4 Ai = pA[t];
            const float4 Bi = pB[t];
            const int dt = t >> 1;
            float px = 0.f, py = 0.f, pzz = 0.f;
            int cnt = 0;
            /* four sources at a time, their LDS loads issued together; the
             * own dumbbell and the sources past the end are masked by a zero
             * 1/r (their term is then exactly zero) */
            for (int j0 = sub; j0 < n; j0 += 4 * split) {
                float4 Aj[4], Bj[4];
                float Fz[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u * split;
                    const int jj = j < n ? j : t;
                    Aj[u] = pA[jj];
                    Bj[u] = pB[jj];
                    Fz[u] = pz[jj];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u * split;
                    float rx, ry, rz;
                    if (SPLIT) {
                        rx = (Ai.x - Aj[u].x) + (Bi.x - Bj[u].x);
                        ry = (Ai.y - Aj[u].y) + (Bi.y - Bj[u].y);
                        rz = (Ai.z - Aj[u].z) + (Bi.z - Bj[u].z);
                    } else {
                        rx = Ai.x - Aj[u].x;
                        ry = Ai.y - Aj[u].y;
                        rz = Ai.z - Aj[u].z;
                    }
                    const float r2 = __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
                    float ir = __builtin_amdgcn_rsqf(r2);
                    if (j >= n || (j >> 1) == dt) ir = 0.f;
                    pair_term<RPY>(ir, rx, ry, rz, Aj[u].w, Bj[u].w, Fz[u], crr, px, py, pzz);
                }
                cnt += 4;
                if (cnt == 32) {
                    two_sum_acc(ax, bx, px);
                    two_sum_acc(ay, by, py);
                    two_sum_acc(az, bz, pzz);
                    px = py = pzz = 0.f;
                    cnt = 0;
                }
            }
            two_sum_acc(ax, bx, px);
            two_sum_acc(ay, by, py);
            two_sum_acc(az, bz, pzz);
        }
        float v[6] = {ax, bx, ay, by, az, bz};
        if (split > 1) combine_level_dpp<0xB1>(v);
        if (split > 2) combine_level_dpp<0x4E>(v);
        for (int sh = 4; sh < split; sh *= 2) combine_level_shfl(v, sh);
        if (own) {
            const double acc[3] = {(double)v[0] + (double)v[1], (double)v[2] + (double)v[3],
                                   (double)v[4] + (double)v[5]};
            for (int a = 0; a < 3; ++a) {
                const double k = u0[a] + c.co * acc[a];
                if (!isfinite(k)) bad = 1;
                const double nz = INTEG == 2 ? c.g * gauss_component(c.seed, ioff + t, step, a) : 0.0;
                y[a] = res_update(c, INTEG == 0 ? 0 : 1, stage, NST, k, x[a], r[a], nz);
            }
        }
        buf ^= 1;
        forces(tb[2 * stage], tb[2 * stage + 1], buf);
    };
    for (int sn = 0; sn < nsteps; ++sn) {
        const long long step = step0 + sn;
        row = row + 1 == d.ring ? 0 : row + 1;
        if (own)
            for (int q = 0; q < 8; ++q) nb[q] = d.tab[row * 8 + q];
        stage_pass(std::integral_constant<int, 0>{}, step);
        stage_pass(std::integral_constant<int, 1>{}, step);
        if constexpr (NST == 4) {
            stage_pass(std::integral_constant<int, 2>{}, step);
            stage_pass(std::integral_constant<int, 3>{}, step);
        }
        for (int q = 0; q < 8; ++q) tb[q] = nb[q];
    }
    if (own)
        for (int a = 0; a < 3; ++a) d.X[a * N + ioff + t] = x[a];
    if (__syncthreads_or(bad) && tid == 0) atomicOr(&d.ctl->flag, FLAG_NONFINITE);
}

/* ------------------------------------------------------------ launchers */

static inline dim3 blocks_for(int n, int bs) { return dim3((unsigned)((n + bs - 1) / bs)); }

hipError_t launch_set_step(const Dev& d, long long step, hipStream_t s) {
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(1), 0, s, d.ctl, step);
    return hipGetLastError();
}

hipError_t launch_clear_flag(const Dev& d, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, s, d.ctl);
    return hipGetLastError();
}

hipError_t launch_clear_counts(const Dev& d, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_counts, blocks_for(d.Ntot, 256), dim3(256), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_state_in(const Dev& d, const double* Xa, hipStream_t s) {
    hipLaunchKernelGGL(k_state_in, blocks_for(d.Ntot, 256), dim3(256), 0, s, d, Xa);
    return hipGetLastError();
}

hipError_t launch_state_out(const Dev& d, double* Xa, hipStream_t s) {
    hipLaunchKernelGGL(k_state_out, blocks_for(d.Ntot, 256), dim3(256), 0, s, d, Xa);
    return hipGetLastError();
}

/* Spheres per wave in the full steric sums (add_steric), 0 where a thread
 * takes a dumbbell: the thread's chain is 0.28 us per sphere of its system,
 * the wave's work 0.0006 us per dumbbell, so from about 1000 systems on the
 * threads are faster, whatever the systems' size, and for one or two dumbbells
 * a system always (64 dumbbells, FP64 step, 36 us and 38; ad_forces, us, thread and
 * wave: 512 systems of 8 spheres 10 and 10, of 200 73 and 35; 8192 of 8 13 and
 * 16; 30000 of 4 10 and 26; a single one of 4096 spheres 1174 and 19). Eight
 * spheres share a wave's loads of a source where that leaves enough waves:
 * 4096 spheres 28 us (two: 19), 16384 119 (145), 65536 1.49 ms (2.28; by
 * threads 18.8). */
static int steric_spheres(const Dev& d, const Coef& c) {
    if (c.ks == 0.0 || d.nsys >= 1024 || d.Ntot <= 4 * d.nsys) return 0;
    return d.nsys == 1 && d.Ntot >= 16384 ? 8 : 2;
}
static dim3 steric_grid(const Dev& d, int it) {
    return it ? blocks_for(d.Stot, 4 * (it / 2)) : blocks_for(d.Stot, 128);
}

hipError_t launch_pack_state(const Dev& d, const Coef& c, int prec, double st, double ct, hipStream_t s) {
    const int it = steric_spheres(d, c);
    const dim3 g = steric_grid(d, it), t(it ? 256 : 128);
    if (it == 0)
        hipLaunchKernelGGL(k_pack_state<0>, g, t, 0, s, d, c, prec, st, ct);
    else if (it == 2)
        hipLaunchKernelGGL(k_pack_state<2>, g, t, 0, s, d, c, prec, st, ct);
    else
        hipLaunchKernelGGL(k_pack_state<8>, g, t, 0, s, d, c, prec, st, ct);
    return hipGetLastError();
}

hipError_t launch_pack_apply(const Dev& d, const Coef& c, int prec, const double* Xa, const double* Fa,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_pack_apply, blocks_for(d.Stot, 128), dim3(128), 0, s, d, c, prec, Xa, Fa);
    return hipGetLastError();
}

hipError_t launch_forces(const Dev& d, const Coef& c, const double* Xa, double st, double ct, double* Fa,
                         hipStream_t s) {
    const int it = steric_spheres(d, c);
    const dim3 g = steric_grid(d, it), t(it ? 256 : 128);
    if (it == 0)
        hipLaunchKernelGGL(k_forces<0>, g, t, 0, s, d, c, Xa, st, ct, Fa);
    else if (it == 2)
        hipLaunchKernelGGL(k_forces<2>, g, t, 0, s, d, c, Xa, st, ct, Fa);
    else
        hipLaunchKernelGGL(k_forces<8>, g, t, 0, s, d, c, Xa, st, ct, Fa);
    return hipGetLastError();
}

/* Launch a pair kernel; with timing events the launch goes through
 * hipExtLaunchKernelGGL, whose events carry the dispatch's own start and end
 * times. */
struct Timing {
    hipEvent_t start, stop;
};

template <class K>
static hipError_t go(K kern, int wg, const Dev& d, const Epi& e, int mode, hipStream_t s, const Timing& tm) {
    if (tm.start)
        hipExtLaunchKernelGGL(kern, dim3(d.nitems), dim3(wg), 0, s, tm.start, tm.stop, 0, d, e, mode);
    else
        hipLaunchKernelGGL(kern, dim3(d.nitems), dim3(wg), 0, s, d, e, mode);
    return hipGetLastError();
}

template <int WG, int WJ, int SPLIT, int STERIC, int RPY>
static hipError_t f32c_ipl(const Dev& d, const Epi& e, int ipl, int mode, hipStream_t s, const Timing& tm) {
    if (ipl == 1) return go(k_pairs_f32c<WG, 1, WJ, SPLIT, STERIC, RPY>, WG, d, e, mode, s, tm);
    if (ipl == 2) return go(k_pairs_f32c<WG, 2, WJ, SPLIT, STERIC, RPY>, WG, d, e, mode, s, tm);
    if (ipl == 4) return go(k_pairs_f32c<WG, 4, WJ, SPLIT, STERIC, RPY>, WG, d, e, mode, s, tm);
    return hipErrorInvalidValue;
}

template <int WG, int WJ, int RPY>
static hipError_t f32c_var(const Dev& d, const Epi& e, const Shape& sh, int mode, hipStream_t s, const Timing& tm) {
    if (sh.steric)
        return sh.split ? f32c_ipl<WG, WJ, 1, 1, RPY>(d, e, sh.ipl, mode, s, tm)
                        : f32c_ipl<WG, WJ, 0, 1, RPY>(d, e, sh.ipl, mode, s, tm);
    return sh.split ? f32c_ipl<WG, WJ, 1, 0, RPY>(d, e, sh.ipl, mode, s, tm)
                    : f32c_ipl<WG, WJ, 0, 0, RPY>(d, e, sh.ipl, mode, s, tm);
}

template <int WG, int WJ>
static hipError_t f32c_ten(const Dev& d, const Epi& e, const Shape& sh, int mode, hipStream_t s, const Timing& tm) {
    return sh.rpy ? f32c_var<WG, WJ, 1>(d, e, sh, mode, s, tm) : f32c_var<WG, WJ, 0>(d, e, sh, mode, s, tm);
}

template <int WG, int IPL>
static hipError_t f64_ten(const Dev& d, const Epi& e, const Shape& sh, int mode, hipStream_t s, const Timing& tm) {
    return sh.rpy ? go(k_pairs_f64<WG, IPL, 1>, WG, d, e, mode, s, tm) : go(k_pairs_f64<WG, IPL, 0>, WG, d, e, mode, s, tm);
}

template <int IPL, int G>
static hipError_t go_f64t(const Dev& d, const Epi& e, const Shape& sh, int mode, hipStream_t s, const Timing& tm) {
    const int per_item = sh.wg / 64;
    const dim3 grid(d.nitems * per_item), block(64 * G);
    auto kern = sh.rpy ? k_pairs_f64t<G, IPL, 1> : k_pairs_f64t<G, IPL, 0>;
    if (tm.start)
        hipExtLaunchKernelGGL(kern, grid, block, 0, s, tm.start, tm.stop, 0, d, e, mode, per_item);
    else
        hipLaunchKernelGGL(kern, grid, block, 0, s, d, e, mode, per_item);
    return hipGetLastError();
}

/* RPY: whether the shape is taken with the correction too */
template <int TW, int NP, int CW, int RPY = 1>
static hipError_t go_f64w(const Dev& d, const Epi& e, const Shape& sh, int mode, hipStream_t s, const Timing& tm) {
    auto kern = RPY && sh.rpy ? k_pairs_f64w<TW, NP, CW, RPY> : k_pairs_f64w<TW, NP, CW, 0>;
    const size_t lds = f64w_lds_bytes({TW, NP, CW}, sh.rpy);
    const dim3 block(64 * (NP + 1));
    if (tm.start)
        hipExtLaunchKernelGGL(kern, dim3(d.nfitems), block, lds, s, tm.start, tm.stop, 0, d, e, mode);
    else
        hipLaunchKernelGGL(kern, dim3(d.nfitems), block, lds, s, d, e, mode);
    return hipGetLastError();
}

hipError_t launch_pairs(const Dev& d, const Epi& e, const Shape& sh, int mode, hipStream_t s, hipEvent_t ev_start,
                        hipEvent_t ev_stop) {
    if (d.nitems <= 0) return hipSuccess;
    const Timing tm{ev_start, ev_stop};
    if (e.prec == PREC_FP32C) {
        if (sh.steric && !d.nbr_cnt) return hipErrorInvalidValue;
        if (sh.wg == 64 && sh.wj == 1) return f32c_ten<64, 1>(d, e, sh, mode, s, tm);
        if (sh.wg == 256 && sh.wj == 1) return f32c_ten<256, 1>(d, e, sh, mode, s, tm);
        if (sh.wg == 256 && sh.wj == 4) return f32c_ten<256, 4>(d, e, sh, mode, s, tm);
        return hipErrorInvalidValue;
    }
    /* AD_FP64: the terms spread over waves (work list of target blocks) */
    if (e.prec == PREC_FP64 && d.f64_blocks && d.nfitems > 0) {
        const F64WShape f = f64w_shape(d.Ntot, sh.rpy, d.nsys);
        if (f.tw == 4 && f.np == 2 && f.cw == 64) return go_f64w<4, 2, 64>(d, e, sh, mode, s, tm);
        if (f.tw == 4 && f.np == 1 && f.cw == 64) return go_f64w<4, 1, 64>(d, e, sh, mode, s, tm);
        if (f.tw == 4 && f.np == 1 && f.cw == 128 && !sh.rpy) return go_f64w<4, 1, 128, 0>(d, e, sh, mode, s, tm);
        if (f.tw == 2 && f.np == 2 && f.cw == 64) return go_f64w<2, 2, 64>(d, e, sh, mode, s, tm);
        if (f.tw == 2 && f.np == 1 && f.cw == 128) return go_f64w<2, 1, 128>(d, e, sh, mode, s, tm);
        return hipErrorInvalidValue;
    }
    /* FP64 kernels: 1 or 2 targets per lane, no j split inside a group; the
     * work list was built for this shape, so anything else is refused */
    if (sh.wj != 1 || (sh.wg != 64 && sh.wg != 256)) return hipErrorInvalidValue;
    if (e.prec == PREC_FP64_TILED) {
        /* one wave per 64 targets where a system's sources are one wave's
         * (4096 systems of 16 spheres 69 us per RK4 step, with four 98; 30000
         * dumbbells 108, 252) */
        const bool small = d.nsys > 1 && d.Ntot / d.nsys <= 64;
        if (sh.ipl == 1) return small ? go_f64t<1, 1>(d, e, sh, mode, s, tm) : go_f64t<1, 4>(d, e, sh, mode, s, tm);
        if (sh.ipl == 2) return small ? go_f64t<2, 1>(d, e, sh, mode, s, tm) : go_f64t<2, 4>(d, e, sh, mode, s, tm);
        return hipErrorInvalidValue;
    }
    if (sh.wg == 64 && sh.ipl == 1) return f64_ten<64, 1>(d, e, sh, mode, s, tm);
    if (sh.wg == 64 && sh.ipl == 2) return f64_ten<64, 2>(d, e, sh, mode, s, tm);
    if (sh.wg == 256 && sh.ipl == 1) return f64_ten<256, 1>(d, e, sh, mode, s, tm);
    if (sh.wg == 256 && sh.ipl == 2) return f64_ten<256, 2>(d, e, sh, mode, s, tm);
    return hipErrorInvalidValue;
}

template <int SPLIT, int RPY, int NW>
static hipError_t go_fused(const Dev& d, const Epi& e, int maxNb, hipStream_t s, const Timing& tm) {
    const int lds = fused_lds_bytes(maxNb, SPLIT, NW);
    const dim3 grid(d.nfitems ? d.nfitems : (d.Ntot + FS_I - 1) / FS_I);
    auto kern = k_stage_fused<SPLIT, RPY, NW>;
    if (tm.start)
        hipExtLaunchKernelGGL(kern, grid, dim3(64 * NW), lds, s, tm.start, tm.stop, 0, d, e);
    else
        hipLaunchKernelGGL(kern, grid, dim3(64 * NW), lds, s, d, e);
    return hipGetLastError();
}

template <int SPLIT, int RPY>
static hipError_t go_wide(const Dev& d, const Epi& e, int maxNb, hipStream_t s, const Timing& tm) {
    const int lds = fused_wide_lds_bytes(maxNb, SPLIT);
    auto kern = k_stage_wide<SPLIT, RPY>;
    if (tm.start)
        hipExtLaunchKernelGGL(kern, dim3(d.nfitems), dim3(256), lds, s, tm.start, tm.stop, 0, d, e);
    else
        hipLaunchKernelGGL(kern, dim3(d.nfitems), dim3(256), lds, s, d, e);
    return hipGetLastError();
}

typedef void (*StageKernel)(Dev, Epi);

template <int SPLIT, int RPY, int NOISE>
static StageKernel stream_kernel(int ti, int x2) {
    if (ti == 16) return x2 ? k_stage_stream_x2<SPLIT, RPY, 16, 16, NOISE> : k_stage_stream<SPLIT, RPY, 16, 16, NOISE>;
    return ti == 8 ? k_stage_stream<SPLIT, RPY, 8, 8, NOISE> : k_stage_stream<SPLIT, RPY, 4, 8, NOISE>;
}
static StageKernel stream_kernel(int split, int rpy, int noise, int ti, int x2) {
    switch (split * 4 + rpy * 2 + noise) {
        case 0: return stream_kernel<0, 0, 0>(ti, x2);
        case 1: return stream_kernel<0, 0, 1>(ti, x2);
        case 2: return stream_kernel<0, 1, 0>(ti, x2);
        case 3: return stream_kernel<0, 1, 1>(ti, x2);
        case 4: return stream_kernel<1, 0, 0>(ti, x2);
        case 5: return stream_kernel<1, 0, 1>(ti, x2);
        case 6: return stream_kernel<1, 1, 0>(ti, x2);
        default: return stream_kernel<1, 1, 1>(ti, x2);
    }
}

static hipError_t go_stream(const Dev& d, const Epi& e, const Shape& sh, hipStream_t s, const Timing& tm) {
    const int ti = stream_targets(d.Ntot), nw = stream_waves(ti);
    const int lds = fused_stream_lds_bytes(sh.split, nw, ti);
    const dim3 grid(d.nfitems ? d.nfitems : (d.Ntot + ti - 1) / ti);
    auto kern = stream_kernel(sh.split ? 1 : 0, sh.rpy ? 1 : 0, e.c.noise ? 1 : 0, ti, grid.x > 256);
    if (tm.start)
        hipExtLaunchKernelGGL(kern, grid, dim3(64 * nw), lds, s, tm.start, tm.stop, 0, d, e);
    else
        hipLaunchKernelGGL(kern, grid, dim3(64 * nw), lds, s, d, e);
    return hipGetLastError();
}

template <int RPY>
static hipError_t go_stream64(const Dev& d, const Epi& e, hipStream_t s, const Timing& tm) {
    const int lds = fused_stream64_lds_bytes();
    const int ti = stream_targets(d.Ntot);
    const dim3 grid(d.nfitems ? d.nfitems : (d.Ntot + ti - 1) / ti);
    auto kern = ti == 16 ? k_stage_stream64<RPY, 16> : ti == 8 ? k_stage_stream64<RPY, 8> : k_stage_stream64<RPY, 4>;
    if (tm.start)
        hipExtLaunchKernelGGL(kern, grid, dim3(1024), lds, s, tm.start, tm.stop, 0, d, e);
    else
        hipLaunchKernelGGL(kern, grid, dim3(1024), lds, s, d, e);
    return hipGetLastError();
}

typedef void (*ResidentKernel)(Dev, Epi, long long, int, double, double);

template <int SPLIT, int RPY, int T>
static ResidentKernel resident_c_integ(int integ) {
    if (integ == 0) return k_resident_c<SPLIT, RPY, T, 0>;
    if (integ == 1) return k_resident_c<SPLIT, RPY, T, 1>;
    return k_resident_c<SPLIT, RPY, T, 2>;
}

template <int T>
static ResidentKernel resident_c_threads(int hilo, int rpy, int integ) {
    if (hilo) return rpy ? resident_c_integ<1, 1, T>(integ) : resident_c_integ<1, 0, T>(integ);
    return rpy ? resident_c_integ<0, 1, T>(integ) : resident_c_integ<0, 0, T>(integ);
}

template <int ONE>
static ResidentKernel resident_form(int rpy, int integ) {
    if (rpy) return integ == 0 ? k_resident<1, 0, ONE> : integ == 1 ? k_resident<1, 1, ONE> : k_resident<1, 2, ONE>;
    return integ == 0 ? k_resident<0, 0, ONE> : integ == 1 ? k_resident<0, 1, ONE> : k_resident<0, 2, ONE>;
}
/* The FP64 resident kernel with the form of up to 16 spheres (one) or without. */
static ResidentKernel resident_kernel(int one, int rpy, int integ) {
    return one ? resident_form<1>(rpy, integ) : resident_form<0>(rpy, integ);
}
/* Which of the two. By their registers a compute unit holds with[] and
 * without[] work-groups of them (or what LDS allows, if fewer). While every
 * system is resident at once with the form, it is the faster one; beyond that
 * it costs another round of work-groups where the other kernel needs none. Up
 * to 8 spheres, whose pairs are one wave, it also pays for as many rounds as
 * the other takes (up to 4 spheres for two). us per RK4 step, Oseen, with and
 * without: 1024 systems of 10 spheres 5.67, 5.82, 1025 8.77, 6.63, 1536 10.5,
 * 9.9, 4096 22.4, 20.3; of 6, 4096 18.9, 20.6; of 4, 1024 4.55, 5.22, 1280 8.70,
 * 6.23, 1400 8.64, 10.5, 4096 19.4, 19.9; of 2, 4096 19.5, 18.7. */
static bool resident_one(int rpy, int integ, int nsys, int maxNb, size_t lds) {
    static const int with[2][3] = {{4, 5, 3}, {4, 4, 3}}, without[2][3] = {{5, 7, 4}, {4, 5, 4}};
    const int by_lds = lds ? (int)(FUSED_LDS_MAX / lds) : 8;
    const int w = 256 * std::min(with[rpy][integ], by_lds), o = 256 * std::min(without[rpy][integ], by_lds);
    if (o <= w || nsys <= w) return true;
    if (maxNb <= 4 && nsys > 2 * w) return false;
    return maxNb <= 8 && (nsys + w - 1) / w <= (nsys + o - 1) / o;
}

/* the FP32C resident kernel for hi/lo positions or not, RPY or not, T
 * threads (64, 128, 256 or 512) and integrator integ (0 RK4, 1 Heun, 2 Heun
 * with noise) */
static ResidentKernel resident_c_kernel(int hilo, int rpy, int T, int integ) {
    switch (T) {
        case 64: return resident_c_threads<64>(hilo, rpy, integ);
        case 128: return resident_c_threads<128>(hilo, rpy, integ);
        case 256: return resident_c_threads<256>(hilo, rpy, integ);
        default: return resident_c_threads<512>(hilo, rpy, integ);
    }
}

hipError_t prepare_fused() {
    const void* kernels[] = {
                             reinterpret_cast<const void*>(&k_stage_stream64<0, 16>),
                             reinterpret_cast<const void*>(&k_stage_stream64<1, 16>),
                             reinterpret_cast<const void*>(&k_stage_stream64<0, 8>),
                             reinterpret_cast<const void*>(&k_stage_stream64<1, 8>),
                             reinterpret_cast<const void*>(&k_stage_stream64<0, 4>),
                             reinterpret_cast<const void*>(&k_stage_stream64<1, 4>),
                             reinterpret_cast<const void*>(&k_stage_wide<0, 0>),
                             reinterpret_cast<const void*>(&k_stage_wide<0, 1>),
                             reinterpret_cast<const void*>(&k_stage_wide<1, 0>),
                             reinterpret_cast<const void*>(&k_stage_wide<1, 1>),
                             reinterpret_cast<const void*>(&k_stage_fused<0, 0, 16>),
                             reinterpret_cast<const void*>(&k_stage_fused<0, 1, 16>),
                             reinterpret_cast<const void*>(&k_stage_fused<1, 0, 16>),
                             reinterpret_cast<const void*>(&k_stage_fused<1, 1, 16>),
                             reinterpret_cast<const void*>(&k_stage_fused<0, 0, 4>),
                             reinterpret_cast<const void*>(&k_stage_fused<0, 1, 4>),
                             reinterpret_cast<const void*>(&k_stage_fused<1, 0, 4>),
                             reinterpret_cast<const void*>(&k_stage_fused<1, 1, 4>)};
    const void* stream[32];
    for (int q = 0; q < 32; ++q) /* hi/lo, RPY, noise; 16 targets with and without the cap, 8, 4 */
        stream[q] = reinterpret_cast<const void*>(
            stream_kernel(q & 1, (q >> 1) & 1, (q >> 2) & 1, q < 16 ? 16 : q < 24 ? 8 : 4, q < 8));
    for (const void* k : stream) {
        hipError_t err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, FUSED_LDS_MAX);
        if (err != hipSuccess) {
            (void)hipGetLastError();
            return err;
        }
    }
    for (const void* k : kernels) {
        hipError_t err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, FUSED_LDS_MAX);
        if (err != hipSuccess) {
            (void)hipGetLastError(); /* a later launch check must not report it again */
            return err;
        }
    }
    const void* resident[60];
    for (int q = 0; q < 12; ++q)
        resident[q] = reinterpret_cast<const void*>(resident_kernel(q & 1, (q >> 1) & 1, q >> 2));
    for (int q = 0; q < 48; ++q)
        resident[12 + q] = reinterpret_cast<const void*>(
            resident_c_kernel(q & 1, (q >> 1) & 1, 64 << ((q >> 2) & 3), q >> 4));
    for (const void* k : resident) {
        hipError_t err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, RES_LDS_MAX);
        if (err != hipSuccess) {
            (void)hipGetLastError();
            return err;
        }
    }
    return hipSuccess;
}

hipError_t launch_resident(const Dev& d, const Epi& e, int hilo, int maxNb, long long step0, int nsteps,
                           double st0, double ct0, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
    if (d.nfitems <= 0 || nsteps <= 0) return hipErrorInvalidValue;
    const int p64 = e.prec != PREC_FP32C;
    const int rpy = e.c.rpy;
    if (maxNb > (p64 ? RES_MAX64 : RES_MAX32)) return hipErrorInvalidValue;
    const size_t lds = (size_t)resident_lds_bytes(maxNb, p64, rpy);
    if (lds > (size_t)RES_LDS_MAX) return hipErrorInvalidValue;
    const int T = resident_threads(maxNb, p64);
    ResidentKernel kern;
    const int integ = e.integ == 0 ? 0 : (e.c.noise ? 2 : 1);
    if (p64)
        kern = resident_kernel(resident_one(rpy, integ, d.nfitems, maxNb, lds), rpy, integ);
    else
        kern = resident_c_kernel(hilo, rpy, T, integ);
    if (ev_start)
        hipExtLaunchKernelGGL(kern, dim3(d.nfitems), dim3(T), lds, s, ev_start, ev_stop, 0, d, e, step0, nsteps, st0,
                              ct0);
    else
        hipLaunchKernelGGL(kern, dim3(d.nfitems), dim3(T), lds, s, d, e, step0, nsteps, st0, ct0);
    return hipGetLastError();
}

hipError_t launch_fused(const Dev& d, const Epi& e, const Shape& sh, int maxNb, hipStream_t s,
                        hipEvent_t ev_start, hipEvent_t ev_stop) {
    const Timing tm0{ev_start, ev_stop};
    if (e.prec == PREC_FP64_TILED && sh.fused == 3 && !sh.steric && maxNb >= 2) {
        if ((d.nsys > 1) != (d.nfitems > 0)) return hipErrorInvalidValue;
        return sh.rpy ? go_stream64<1>(d, e, s, tm0) : go_stream64<0>(d, e, s, tm0);
    }
    if (e.prec != PREC_FP32C || sh.steric || maxNb < 2) return hipErrorInvalidValue;
    if (sh.fused == 2) {
        /* every work-group takes its (system, 64-target block) from the list */
        if (d.nfitems <= 0 || fused_wide_lds_bytes(maxNb, sh.split) > FUSED_LDS_MAX) return hipErrorInvalidValue;
        if (sh.split) return sh.rpy ? go_wide<1, 1>(d, e, maxNb, s, tm0) : go_wide<1, 0>(d, e, maxNb, s, tm0);
        return sh.rpy ? go_wide<0, 1>(d, e, maxNb, s, tm0) : go_wide<0, 0>(d, e, maxNb, s, tm0);
    }
    if ((d.nsys > 1) != (d.nfitems > 0)) return hipErrorInvalidValue;
    if (sh.fused == 3) return go_stream(d, e, sh, s, tm0);
    if (sh.fused != 1) return hipErrorInvalidValue;
    const int nw = d.nsys > 1 ? 4 : 16;
    if (fused_lds_bytes(maxNb, sh.split, nw) > FUSED_LDS_MAX) return hipErrorInvalidValue;
    const Timing tm{ev_start, ev_stop};
    if (nw == 16) {
        if (sh.split) return sh.rpy ? go_fused<1, 1, 16>(d, e, maxNb, s, tm) : go_fused<1, 0, 16>(d, e, maxNb, s, tm);
        return sh.rpy ? go_fused<0, 1, 16>(d, e, maxNb, s, tm) : go_fused<0, 0, 16>(d, e, maxNb, s, tm);
    }
    if (sh.split) return sh.rpy ? go_fused<1, 1, 4>(d, e, maxNb, s, tm) : go_fused<1, 0, 4>(d, e, maxNb, s, tm);
    return sh.rpy ? go_fused<0, 1, 4>(d, e, maxNb, s, tm) : go_fused<0, 0, 4>(d, e, maxNb, s, tm);
}

hipError_t launch_epilogue(const Dev& d, const Epi& e, hipStream_t s) {
    if (pairs_close(d, e)) return hipSuccess;
    hipLaunchKernelGGL(k_epilogue, blocks_for(d.Ntot, EPI_S), dim3(EPI_T), 0, s, d, e);
    return hipGetLastError();
}

hipError_t launch_steric_pack(const Dev& d, const Coef& c, int prec, hipStream_t s) {
    const int it = d.nbr_cnt ? 0 : steric_spheres(d, c);
    const dim3 g = steric_grid(d, it), t(it ? 256 : 128);
    if (d.nbr_cnt)
        hipLaunchKernelGGL((k_steric_pack<1, 0>), g, t, 0, s, d, c, prec);
    else if (it == 0)
        hipLaunchKernelGGL((k_steric_pack<0, 0>), g, t, 0, s, d, c, prec);
    else if (it == 2)
        hipLaunchKernelGGL((k_steric_pack<0, 2>), g, t, 0, s, d, c, prec);
    else
        hipLaunchKernelGGL((k_steric_pack<0, 8>), g, t, 0, s, d, c, prec);
    return hipGetLastError();
}

hipError_t launch_record(const Dev& d, int maxNb, double* centres, double* com, hipStream_t s) {
    const bool threads = d.nsys / 64 >= maxNb;
    const int ncom = !com ? 0 : threads ? (3 * d.nsys + REC_WG - 1) / REC_WG : d.nsys;
    const int ncen = centres ? (d.Stot + REC_WG - 1) / REC_WG : 0;
    if (ncom + ncen == 0) return hipSuccess;
    hipLaunchKernelGGL(threads ? k_record<1> : k_record<0>, dim3(ncom + ncen), dim3(REC_WG), 0, s, d, centres, com,
                       ncom);
    return hipGetLastError();
}

}  // namespace ad
