/*
 * Stroke-averaged far-field equations of motion on gfx950 (Putz, Dunkel,
 * Yeomans, Sec. III, Eqs. e:eom, J, K and the projections s, r, q):
 *   dR_s/dt = sum_{r != s} J^{sr},   dN_s/dt = -(I - N_s N_s) sum_{r != s} K^{sr},
 *   J^{sr} = a w sin(phi_s - phi_r) (9/64) (lam/ell)^2 (ell/D)^4
 *            { N_s (2s + 4qr - 10 s r^2)
 *              + Dhat (1 + 2q^2 - 5s^2 - 5r^2 - 20 q s r + 35 s^2 r^2) },
 *   K^{sr} = w sin(phi_s - phi_r) (15/64) (a/ell) (lam/ell)^2 (ell/D)^5 Dhat
 *            (3s + 6rq + 6 s q^2 - 7 s^3 - 21 s r^2 - 42 q s^2 r + 63 s^3 r^2),
 *   D = R_s - R_r, s = Dhat.N_s, r = Dhat.N_r, q = N_s.N_r.
 * One dumbbell per WPT waves: the lanes share the sum over the others, a
 * fixed butterfly and, with WPT = 4, the waves' sums through LDS in a fixed
 * order add the partial sums. FP64 throughout, FMAs written out. With up to
 * SA_WIDE dumbbells the launch has fewer waves than the chip has SIMDs at one
 * wave per dumbbell, and a stage is a chain of latencies (loads, the terms
 * one after another, the reduction, the update): four waves per dumbbell
 * shorten the terms' part. Above that what bounds a stage is FP64 issue,
 * about 80 instructions per pair (reciprocal square root, a sine over one
 * period, Horner forms of the three polynomials), where the plain form's
 * square root, four divisions and library sine took about 250.
 * Per RK4 step: 343 dumbbells 24.7 us (39 in the plain form with one wave per
 * dumbbell; k_sa_stage 5.2 us against 9.4), 4096 dumbbells 263 us (531). The
 * rates' error against 80 bits (root mean square over 27 to 800 dumbbells,
 * six draws each): 0.80e-15 and 0.87e-15 against 0.79e-15 and 0.91e-15.
 * A step is four launches of k_sa_stage (RK4); each also applies its stage's
 * update to its own dumbbell, and the last one scales the axes back to unit
 * length.
 */
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/ad.h"

namespace ad_sa {

constexpr double kPi = 3.14159265358979323846;
constexpr int SA_WG = 256;   /* 4 / WPT dumbbells */
constexpr int SA_WIDE = 1024; /* four waves per dumbbell up to this many, one above */

struct SaCoef {
    double ell, cj, ck; /* cj = a w (9/64)(lam/ell)^2, ck = w (15/64)(a/ell)(lam/ell)^2 */
    double h2, dt, dt6;
};

__device__ __forceinline__ unsigned sa_hi(double x) {
    return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32);
}

/* sin x for |x| < 2^19: reduced by the nearest multiple n of pi (pi as the sum
 * of two doubles; the first product-difference is exact), then the odd Taylor
 * polynomial on [-pi/2, pi/2] up to r^21 (the next term is below 2^-59), with
 * the sign (-1)^n. Within an ulp. */
__device__ __forceinline__ double sa_sin(double x) {
    const double n = __builtin_rint(x * 0x1.45f306dc9c883p-2);
    double r = __builtin_fma(-n, 0x1.921fb54442d18p+1, x);
    r = __builtin_fma(-n, 0x1.1a62633145c07p-53, r);
    const double z = r * r;
    double p = 1.0 / 51090942171709440000.0; /* 1/21! */
    p = __builtin_fma(p, z, -1.0 / 121645100408832000.0);
    p = __builtin_fma(p, z, 1.0 / 355687428096000.0);
    p = __builtin_fma(p, z, -1.0 / 1307674368000.0);
    p = __builtin_fma(p, z, 1.0 / 6227020800.0);
    p = __builtin_fma(p, z, -1.0 / 39916800.0);
    p = __builtin_fma(p, z, 1.0 / 362880.0);
    p = __builtin_fma(p, z, -1.0 / 5040.0);
    p = __builtin_fma(p, z, 1.0 / 120.0);
    p = __builtin_fma(p, z, -1.0 / 6.0);
    const double s = __builtin_fma(r * z, p, r);
    const unsigned long long sign = (unsigned long long)((int)n & 1) << 63;
    return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, s) ^ sign);
}

/* 1/sqrt(x), rounded but for rare last-bit cases (the rates hold its fifth
 * power): v_rsq_f64 (about 2^-24) and one third-order step whose residual
 * 1 - x y^2 includes the rounding of x y */
__device__ __forceinline__ double sa_rsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double g = x * y;
    const double e = __builtin_fma(-__builtin_fma(x, y, -g), y, __builtin_fma(-g, y, 1.0));
    return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xF, 0xF, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, false);
    return v + __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
/* sum over the wave, the same bits in every lane: pairs, quads, halves of a
 * row and rows by DPP (a VALU operand modifier), the four rows by exchanges */
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1>(v);  /* quad_perm [1,0,3,2] */
    v = dpp_add<0x4E>(v);  /* quad_perm [2,3,0,1] */
    v = dpp_add<0x141>(v); /* row_half_mirror */
    v = dpp_add<0x140>(v); /* row_mirror */
    v = v + __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

/* The rates of dumbbell i against all S, positions Rs and axes Ns; called by
 * all threads of the work-group, wave w of it working for dumbbell i (i >= S:
 * none). Lane c < 6 of the first wave of i returns component c of (dR, dN);
 * *bad is raised in every lane of that wave when two centres coincide. */
template <int WPT>
__device__ __forceinline__ double sa_rates(const SaCoef& k, int S, int i, const double* __restrict__ Rs,
                                           const double* __restrict__ Ns, const double* __restrict__ phi, int* bad) {
    __shared__ double red[4][8];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, sub = w % WPT;
    double ri[3] = {0.0, 0.0, 0.0}, ni[3] = {0.0, 0.0, 0.0}, pi_ = 0.0;
    if (i < S) {
        for (int a = 0; a < 3; ++a) {
            ri[a] = Rs[3 * i + a];
            ni[a] = Ns[3 * i + a];
        }
        pi_ = phi[i];
    }
    /* the sums of fj aN, fj aD u and fk u; the constants and the axis n_i,
     * common to every term, are applied after the sum */
    double v[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int same = 0;
#pragma unroll 2
    for (int j = sub * 64 + l; j < S; j += 64 * WPT) {
        const double rj[3] = {Rs[3 * j], Rs[3 * j + 1], Rs[3 * j + 2]};
        const double nj[3] = {Ns[3 * j], Ns[3 * j + 1], Ns[3 * j + 2]};
        const double ph = pi_ - phi[j];
        const double Dx = ri[0] - rj[0], Dy = ri[1] - rj[1], Dz = ri[2] - rj[2];
        /* the dumbbell itself: D = 0 at distance 1, weight 0 */
        const bool self = j == i;
        const double D2 = self ? 1.0 : __builtin_fma(Dz, Dz, __builtin_fma(Dy, Dy, Dx * Dx));
        double iD = sa_rsqrt(D2), sn = sa_sin(ph);
        /* operands out of the short forms' range */
        const bool far = sa_hi(D2) - ((1023u - 900u) << 20) >= (1800u << 20);
        if (far || (sa_hi(ph) & 0x7fffffffu) >= ((1023u + 19u) << 20)) {
            const double D = sqrt(D2);
            if (D == 0.0) {
                same = 1;
                continue;
            }
            iD = 1.0 / D;
            sn = sin(ph);
        }
        const double ux = Dx * iD, uy = Dy * iD, uz = Dz * iD;
        const double s = __builtin_fma(uz, ni[2], __builtin_fma(uy, ni[1], ux * ni[0]));
        const double r = __builtin_fma(uz, nj[2], __builtin_fma(uy, nj[1], ux * nj[0]));
        const double q = __builtin_fma(ni[2], nj[2], __builtin_fma(ni[1], nj[1], ni[0] * nj[0]));
        const double x = k.ell * iD, x2 = x * x;
        const double fj = self ? 0.0 : sn * (x2 * x2); /* x is ell there: its fourth power may overflow */
        const double sr = s * r, q2 = q + q;
        /* 2s + 4qr - 10 s r^2 */
        const double aN = __builtin_fma(r, __builtin_fma(-10.0, sr, q2 + q2), s + s);
        /* 1 + 2q^2 - 5s^2 - 5r^2 - 20 q s r + 35 s^2 r^2 */
        double aD = __builtin_fma(q, __builtin_fma(-20.0, sr, q2), 1.0);
        aD = __builtin_fma(-5.0, __builtin_fma(s, s, r * r), aD);
        aD = __builtin_fma(35.0 * sr, sr, aD);
        /* 6rq + s (3 + 6q^2 - 7s^2 - 21r^2 + s r (63 s r - 42 q)) */
        const double q6 = 6.0 * q;
        double c = __builtin_fma(sr, __builtin_fma(63.0, sr, -42.0 * q), 3.0);
        c = __builtin_fma(q6, q, c);
        c = __builtin_fma(-7.0 * s, s, c);
        c = __builtin_fma(-21.0 * r, r, c);
        const double bK = __builtin_fma(s, c, q6 * r);
        const double fD = fj * aD, fk = (fj * x) * bK;
        v[0] = __builtin_fma(fj, aN, v[0]);
        v[1] = __builtin_fma(fD, ux, v[1]);
        v[2] = __builtin_fma(fD, uy, v[2]);
        v[3] = __builtin_fma(fD, uz, v[3]);
        v[4] = __builtin_fma(fk, ux, v[4]);
        v[5] = __builtin_fma(fk, uy, v[5]);
        v[6] = __builtin_fma(fk, uz, v[6]);
    }
#pragma unroll
    for (int a = 0; a < 7; ++a) v[a] = wave_sum(v[a]);
    *bad = __any(same);
    if (WPT > 1) {
        if (l == 0) {
            for (int a = 0; a < 7; ++a) red[w][a] = v[a];
            red[w][7] = *bad ? 1.0 : 0.0;
        }
        __syncthreads();
        if (sub == 0) {
            for (int a = 0; a < 7; ++a) v[a] = (v[a] + red[w + 1][a]) + (red[w + 2][a] + red[w + 3][a]);
            *bad = (red[w][7] + red[w + 1][7]) + (red[w + 2][7] + red[w + 3][7]) != 0.0;
        }
    }
    const int a = l >= 3 ? l - 3 : l;
    const double n_a = a == 0 ? ni[0] : a == 1 ? ni[1] : ni[2];
    if (l < 3) return k.cj * __builtin_fma(n_a, v[0], a == 0 ? v[1] : a == 1 ? v[2] : v[3]);
    const double nk = __builtin_fma(ni[2], v[6], __builtin_fma(ni[1], v[5], ni[0] * v[4]));
    return -(k.ck * __builtin_fma(-n_a, nk, a == 0 ? v[4] : a == 1 ? v[5] : v[6]));
}

template <int WPT>
__global__ __launch_bounds__(SA_WG) void k_sa_rhs(SaCoef k, int S, const double* __restrict__ R,
                                                  const double* __restrict__ N, const double* __restrict__ phi,
                                                  double* __restrict__ dR, double* __restrict__ dN) {
    const int i = blockIdx.x * (4 / WPT) + (threadIdx.x >> 6) / WPT, l = threadIdx.x & 63;
    int bad = 0;
    const double v = sa_rates<WPT>(k, S, i, R, N, phi, &bad);
    if ((threadIdx.x >> 6) % WPT != 0 || i >= S || l >= 6) return;
    (l < 3 ? dR + 3 * i + l : dN + 3 * i + l - 3)[0] = v;
}

/* One RK4 stage: rates at the stage positions (YR, YN), accumulate, and write
 * the next stage positions (or, at the last stage, the new state). */
template <int WPT>
__global__ __launch_bounds__(SA_WG) void k_sa_stage(SaCoef k, int S, int stage, double* __restrict__ R,
                                                    double* __restrict__ N, const double* __restrict__ phi,
                                                    const double* __restrict__ YR, const double* __restrict__ YN,
                                                    double* __restrict__ ZR, double* __restrict__ ZN,
                                                    double* __restrict__ AR, double* __restrict__ AN, int* flag) {
    const int i = blockIdx.x * (4 / WPT) + (threadIdx.x >> 6) / WPT, l = threadIdx.x & 63;
    const bool own = (threadIdx.x >> 6) % WPT == 0 && i < S && l < 6;
    const int o = 3 * i + (l < 3 ? l : l - 3);
    /* the update's inputs, one component per lane, in flight under the sums */
    double x = 0.0, acc = 0.0;
    if (own) {
        x = (l < 3 ? R : N)[o];
        if (stage > 0) acc = (l < 3 ? AR : AN)[o];
    }
    int bad = 0;
    const double v = sa_rates<WPT>(k, S, i, YR, YN, phi, &bad);
    if ((threadIdx.x >> 6) % WPT != 0 || i >= S) return;
    if (bad && l == 0) atomicOr(flag, 1);
    if (stage < 3) {
        if (own) {
            (l < 3 ? AR : AN)[o] = stage == 0 ? v : acc + 2.0 * v;
            (l < 3 ? ZR : ZN)[o] = x + (stage == 2 ? k.dt : k.h2) * v;
        }
        return;
    }
    const double y = x + k.dt6 * (acc + v);
    const double n0 = __shfl(y, 3), n1 = __shfl(y, 4), n2 = __shfl(y, 5);
    if (own) {
        if (l < 3)
            R[o] = y;
        else
            N[o] = y / sqrt((n0 * n0 + n1 * n1) + n2 * n2);
    }
}

__global__ void k_sa_clear(int* flag) { *flag = 0; }

static bool sa_params_ok(const ad_params* p) {
    if (!p) return false;
    const double v[] = {p->a, p->ell, p->lambda, p->T};
    for (double x : v)
        if (!isfinite(x)) return false;
    return p->a > 0 && p->ell > 0 && p->T > 0;
}

static SaCoef sa_coef(const ad_params* p, double dt) {
    SaCoef k;
    const double w = 2.0 * kPi / p->T;
    const double lr = p->lambda / p->ell;
    k.ell = p->ell;
    k.cj = p->a * w * (9.0 / 64.0) * lr * lr;
    k.ck = w * (15.0 / 64.0) * (p->a / p->ell) * lr * lr;
    k.h2 = 0.5 * dt;
    k.dt = dt;
    k.dt6 = dt / 6.0;
    return k;
}

static dim3 sa_grid(int S) { return dim3(S <= SA_WIDE ? S : (S + 3) / 4); }

static size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace ad_sa

using namespace ad_sa;

extern "C" {

int ad_sa_workspace_size(int32_t S, uint64_t* bytes) {
    if (S < 1 || !bytes) return AD_EINVAL;
    /* flag, then YA, YB (R and N each), AR, AN */
    *bytes = 256 + 6 * align256((size_t)S * 3 * sizeof(double));
    return AD_OK;
}

int ad_sa_rhs(const ad_params* p, int32_t S, const double* R, const double* N, const double* phi, double* dR,
              double* dN, void* stream) {
    if (!sa_params_ok(p) || S < 1 || !R || !N || !phi || !dR || !dN) return AD_EINVAL;
    const SaCoef k = sa_coef(p, 1.0);
    hipLaunchKernelGGL(S <= SA_WIDE ? k_sa_rhs<4> : k_sa_rhs<1>, sa_grid(S), dim3(SA_WG), 0, (hipStream_t)stream, k, S,
                       R, N, phi, dR, dN);
    return hipGetLastError() == hipSuccess ? AD_OK : AD_EDEVICE;
}

int ad_sa_run(const ad_params* p, int32_t S, double* R, double* N, const double* phi, double dt, int64_t nsteps,
              void* workspace, uint64_t ws_bytes, void* stream) {
    if (!sa_params_ok(p) || S < 1 || !R || !N || !phi || !(dt > 0) || !isfinite(dt) || nsteps < 0 || !workspace)
        return AD_EINVAL;
    uint64_t need = 0;
    ad_sa_workspace_size(S, &need);
    if (ws_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 256) return AD_ENOMEM;
    hipStream_t st = (hipStream_t)stream;
    char* b = static_cast<char*>(workspace);
    const size_t blk = align256((size_t)S * 3 * sizeof(double));
    int* flag = reinterpret_cast<int*>(b);
    double* YA_R = reinterpret_cast<double*>(b + 256);
    double* YA_N = reinterpret_cast<double*>(b + 256 + blk);
    double* YB_R = reinterpret_cast<double*>(b + 256 + 2 * blk);
    double* YB_N = reinterpret_cast<double*>(b + 256 + 3 * blk);
    double* AR = reinterpret_cast<double*>(b + 256 + 4 * blk);
    double* AN = reinterpret_cast<double*>(b + 256 + 5 * blk);
    const SaCoef k = sa_coef(p, dt);
    const dim3 grid = sa_grid(S), block(SA_WG);
    auto kern = S <= SA_WIDE ? k_sa_stage<4> : k_sa_stage<1>;
    hipLaunchKernelGGL(k_sa_clear, dim3(1), dim3(1), 0, st, flag);
    for (int64_t n = 0; n < nsteps; ++n) {
        /* stage inputs: state, YA, YB, YA; outputs: YA, YB, YA, state */
        hipLaunchKernelGGL(kern, grid, block, 0, st, k, S, 0, R, N, phi, R, N, YA_R, YA_N, AR, AN, flag);
        hipLaunchKernelGGL(kern, grid, block, 0, st, k, S, 1, R, N, phi, YA_R, YA_N, YB_R, YB_N, AR, AN, flag);
        hipLaunchKernelGGL(kern, grid, block, 0, st, k, S, 2, R, N, phi, YB_R, YB_N, YA_R, YA_N, AR, AN, flag);
        hipLaunchKernelGGL(kern, grid, block, 0, st, k, S, 3, R, N, phi, YA_R, YA_N, YB_R, YB_N, AR, AN, flag);
        if (hipGetLastError() != hipSuccess) return AD_EDEVICE;
    }
    int h = 0;
    if (hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess) return AD_EDEVICE;
    if (hipStreamSynchronize(st) != hipSuccess) return AD_EDEVICE;
    return h ? AD_ENONFINITE : AD_OK;
}

}  // extern "C"
