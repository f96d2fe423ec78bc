/*
 * FP32C pair sum of one large system that forms every unordered pair once
 * (k_pairs_sym): r, r^2, 1/r and 1/r^2 are the same for sphere i's term from j
 * and for j's from i, so a pair's two terms share 8 of their 18 instructions
 * (with hi/lo positions 14 of 24).
 *
 * Spheres are cut into blocks of BS = 128 NW and chunks of 64. A work item is
 * a block I and a run of chunks at or above it. Its work-group of NW waves
 * holds the block's spheres in registers, two per lane with their forces and
 * sums, and takes the run's chunks one after another:
 *   - a chunk of a higher block, 64 steps: step 16 g + u pairs lane (row r,
 *     column c) with a sphere of the chunk's row r + g mod 4: the dumbbell of
 *     column c, the next one and so on around the row, its two spheres one
 *     after the other (u = 2m + 0, 1: the lane's own parity first where m is
 *     even, the other first where it is odd). A sum then never carries one
 *     sphere's term of a dumbbell far without the other's, which nearly
 *     cancels it (single steps around the row did, with 1 % more error). The
 *     chunk's spheres are read from LDS, every row twice, so that the steps'
 *     addresses differ by constants; their three partial sums move with them,
 *     by a DPP swap of a pair or rotation of a row by two. After every 16
 *     steps (32 terms) they are folded into a (hi, lo) pair by TwoSum, which
 *     moves a row with them; the lanes' own sums are folded every 64 terms.
 *     The waves' sums of the chunk's spheres are added in wave order through
 *     LDS and go to slot I of their block;
 *   - a chunk of the block itself: the ordered sum, every lane reading the
 *     same sphere, its own dumbbell masked (its terms are in u0, in FP64).
 * At the run's end the lanes' own sums go to the next slot of block I. The
 * epilogue adds a block's slots in order, so the result does not depend on
 * which work-group ran when.
 *
 * With steric forces the running minimum of r^2 over 16 steps is compared
 * with the candidate radius once, and the steps are gone over again only
 * where some pair is closer.
 *
 * What bounds it is VALU issue: 15 instructions per ordered term (18.3 with
 * hi/lo positions) where the ordered sum takes 18.25 (24). 65536 spheres with
 * hi/lo positions and steric forces: 1.6 ms per stage, the ordered sum 2.29.
 */
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "ad_internal.h"

namespace ad {

namespace {

__device__ __forceinline__ void fold(float& hi, float& lo, float v) {
    const float s = hi + v;
    const float bb = s - hi;
    const float e = (hi - (s - bb)) + (v - bb);
    hi = s;
    lo = lo + e;
}

/* x[q] = 1/sqrt(x[q]) (v_rsq_f32), and (qx, qy, qz) from the neighbour in the
 * pair of lanes (ROW = 0) or from two lanes on in the row of 16, the first two
 * after its last (ROW = 1). Both kinds end the issue of two waves' vector
 * instructions at once (see rsq4): together, between two scalar instructions,
 * once per step (65536 spheres hi/lo 6.21 ms per RK4 step, 6.43 with the moves
 * left to the compiler, 6.95 with neither set apart). Moves read registers
 * written two instructions before at the latest, as DPP needs. */
#define AD_MOVE3(CTRL)                                                              \
    "v_mov_b32_dpp %0, %0 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"     \
    "v_mov_b32_dpp %1, %1 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"     \
    "v_mov_b32_dpp %2, %2 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
template <int ROW>
__device__ __forceinline__ void rsq_move(float x[2], float& qx, float& qy, float& qz) {
    if (ROW)
        asm("s_setprio 3\n\tv_rsq_f32 %3, %3\n\tv_rsq_f32 %4, %4\n\t" AD_MOVE3("row_ror:14") "s_setprio 0"
            : "+v"(qx), "+v"(qy), "+v"(qz), "+v"(x[0]), "+v"(x[1]));
    else
        asm("s_setprio 3\n\tv_rsq_f32 %3, %3\n\tv_rsq_f32 %4, %4\n\t" AD_MOVE3("quad_perm:[1,0,3,2]") "s_setprio 0"
            : "+v"(qx), "+v"(qy), "+v"(qz), "+v"(x[0]), "+v"(x[1]));
}
#undef AD_MOVE3

/* What both terms of a pair share. */
template <int RPY>
struct Pair {
    float rx, ry, rz, ir, ir2, av, bw;
    __device__ __forceinline__ void set(float x, float y, float z, float inv, float crr) {
        rx = x; ry = y; rz = z;
        ir = inv;
        ir2 = ir * ir;
        if (RPY) {
            const float ir3 = ir * ir2;
            av = __builtin_fmaf(crr, ir3, ir);
            bw = __builtin_fmaf(-3.0f * crr, ir3, ir);
        }
    }
    /* p += the term of a source with force F (the same expression seen from
     * either end: r enters twice) */
    __device__ __forceinline__ void add(float Fx, float Fy, float Fz, float& px, float& py, float& pz) const {
        const float tt = __builtin_fmaf(rz, Fz, __builtin_fmaf(ry, Fy, rx * Fx)) * ir2;
        if (RPY) {
            const float bv = tt * bw;
            px = __builtin_fmaf(av, Fx, __builtin_fmaf(bv, rx, px));
            py = __builtin_fmaf(av, Fy, __builtin_fmaf(bv, ry, py));
            pz = __builtin_fmaf(av, Fz, __builtin_fmaf(bv, rz, pz));
        } else {
            px = __builtin_fmaf(ir, __builtin_fmaf(tt, rx, Fx), px);
            py = __builtin_fmaf(ir, __builtin_fmaf(tt, ry, Fy), py);
            pz = __builtin_fmaf(ir, __builtin_fmaf(tt, rz, Fz), pz);
        }
    }
};

}  // namespace

template <int NW, int SPLIT, int STERIC, int RPY>
__global__ __launch_bounds__(64 * NW) void k_pairs_sym(Dev d, Epi e) {
    constexpr int IPL = 2, BS = 64 * IPL * NW, W = 16;
    __shared__ float4 sA[2][128];
    __shared__ float4 sB[2][SPLIT ? 128 : 1];
    __shared__ float2 sF[2][128]; /* (Fy, Fz) */
    __shared__ float red[2][NW][6][64];
    advance_slots(d, e);
    const Item it = d.sym_items[blockIdx.x]; /* i0: block's first sphere, j0: first chunk, nj: chunks, c: slot */
    const int N = d.Ntot;
    const int t = threadIdx.x, l = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ib = it.i0 + (w * 64 + l) * IPL;
    const float crr = e.c.crr;

    float hx[IPL], hy[IPL], hz[IPL], lx[IPL], ly[IPL], lz[IPL], fx[IPL], fy[IPL], fz[IPL];
    float px[IPL], py[IPL], pz[IPL], ax[IPL], ay[IPL], az[IPL], bx[IPL], by[IPL], bz[IPL];
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        /* past the end: far away (and far from the chunks' padding), no force */
        float4 A = make_float4(-1.0e15f, -1.0e15f, -1.0e15f, 0.f), B = make_float4(0.f, 0.f, 0.f, 0.f);
        float2 F = make_float2(0.f, 0.f);
        if (ib + q < N) {
            A = d.pA[ib + q];
            if (SPLIT) B = d.pB[ib + q];
            F = d.pC[ib + q];
        }
        hx[q] = A.x; hy[q] = A.y; hz[q] = A.z; fx[q] = A.w; fy[q] = F.x; fz[q] = F.y;
        lx[q] = B.x; ly[q] = B.y; lz[q] = B.z;
        px[q] = py[q] = pz[q] = ax[q] = ay[q] = az[q] = bx[q] = by[q] = bz[q] = 0.f;
    }
    /* the chunk's entries: thread t < 64 holds sphere t of the next chunk */
    float4 eA, eB;
    float2 eF;
    auto fetch = [&](int c) {
        if (t >= 64) return;
        const int j = c * 64 + t;
        eA = make_float4(1.0e15f, 1.0e15f, 1.0e15f, 0.f);
        eB = make_float4(0.f, 0.f, 0.f, 0.f);
        eF = make_float2(0.f, 0.f);
        if (j < N) {
            eA = d.pA[j];
            if (SPLIT) eB = d.pB[j];
            eF = d.pC[j];
        }
    };
    auto put = [&](int b) {
        if (t >= 64) return;
        const int x = (t >> 4) * 32 + (t & 15);
        sA[b][x] = sA[b][x + 16] = eA;
        if (SPLIT) sB[b][x] = sB[b][x + 16] = eB;
        sF[b][x] = sF[b][x + 16] = eF;
    };
    auto separation = [&](int q, const float4& A, const float4& B, float& rx, float& ry, float& rz) {
        if (SPLIT) {
            rx = (hx[q] - A.x) + (lx[q] - B.x);
            ry = (hy[q] - A.y) + (ly[q] - B.y);
            rz = (hz[q] - A.z) + (lz[q] - B.z);
        } else {
            rx = hx[q] - A.x;
            ry = hy[q] - A.y;
            rz = hz[q] - A.z;
        }
        return __builtin_fmaf(rz, rz, __builtin_fmaf(ry, ry, rx * rx));
    };

    fetch(it.j0);
    put(0);
    __syncthreads();
    for (int k = 0; k < it.nj; ++k) {
        const int b = k & 1, c = it.j0 + k;
        if (k + 1 < it.nj) fetch(c + 1);
        const bool own = c * 64 < it.i0 + BS;
        if (own) {
#pragma unroll 2
            for (int v = 0; v < 64; ++v) {
                const int x = (v >> 4) * 32 + (v & 15);
                const float4 A = sA[b][x], B = SPLIT ? sB[b][x] : A;
                const float2 F = sF[b][x];
                const int j = c * 64 + v;
#pragma unroll
                for (int q = 0; q < IPL; ++q) {
                    float rx, ry, rz;
                    const float r2 = separation(q, A, B, rx, ry, rz);
                    if (STERIC && r2 < d.list_r2 && j != ib + q && ib + q < N) {
                        int jr = j;
                        /* j < N is tested here, where few come, not per source: 15000
                         * spheres 91.9 us per launch, 90.1 so */
                        asm volatile("" : "+v"(jr));
                        if (jr < N) append(d.nbr_cnt, d.nbr_idx, &d.ctl->flag, ib + q, jr);
                    }
                    Pair<RPY> pr;
                    pr.set(rx, ry, rz, (j >> 1) == (ib >> 1) ? 0.f : rsq1(r2), crr);
                    pr.add(A.w, F.x, F.y, px[q], py[q], pz[q]);
                }
            }
        } else {
            float qx = 0.f, qy = 0.f, qz = 0.f, cx = 0.f, cy = 0.f, cz = 0.f, gx = 0.f, gy = 0.f, gz = 0.f;
#pragma unroll 1
            for (int s0 = 0; s0 < 4; ++s0) {
                const int row = ((l >> 4) + s0) & 3;
                const int x[2] = {row * 32 + (l & 15), row * 32 + ((l & 15) ^ 1)};
                unsigned rmin = 0x7f800000u; /* the smallest r^2, by its bits (none is negative) */
#pragma unroll
                for (int u = 0; u < W; ++u) {
                    const int at = x[(u ^ (u >> 1)) & 1] + (u & ~1);
                    const float4 A = sA[b][at], B = SPLIT ? sB[b][at] : A;
                    const float2 F = sF[b][at];
                    float rx[IPL], ry[IPL], rz[IPL], ir[IPL];
#pragma unroll
                    for (int q = 0; q < IPL; ++q) ir[q] = separation(q, A, B, rx[q], ry[q], rz[q]);
                    if (STERIC) {
                        rmin = min(rmin, min(__builtin_bit_cast(unsigned, ir[0]), __builtin_bit_cast(unsigned, ir[1])));
                        asm volatile("" : "+v"(rmin));
                    }
                    if (u & 1) {
                        rsq_move<0>(ir, qx, qy, qz);
                    } else if (u > 0) {
                        rsq_move<1>(ir, qx, qy, qz);
                    } else {
                        ir[0] = rsq1(ir[0]);
                        ir[1] = rsq1(ir[1]);
                    }
#pragma unroll
                    for (int q = 0; q < IPL; ++q) {
                        Pair<RPY> pr;
                        pr.set(rx[q], ry[q], rz[q], ir[q], crr);
                        pr.add(A.w, F.x, F.y, px[q], py[q], pz[q]);
                        pr.add(fx[q], fy[q], fz[q], qx, qy, qz);
                    }
                    /* each step's sums are formed in it: left alone, the
                     * compiler puts off one side of all 16 steps and
                     * keeps their separations in 260 registers */
                    asm volatile("" : "+v"(qx), "+v"(qy), "+v"(qz), "+v"(px[0]), "+v"(py[0]), "+v"(pz[0]),
                                 "+v"(px[1]), "+v"(py[1]), "+v"(pz[1]));
                }
                /* the folded sums follow the partial ones, a row at a time */
                if (s0 > 0) {
                    const int from = (l + 16) & 63;
                    cx = __shfl(cx, from); cy = __shfl(cy, from); cz = __shfl(cz, from);
                    gx = __shfl(gx, from); gy = __shfl(gy, from); gz = __shfl(gz, from);
                }
                fold(cx, gx, qx);
                fold(cy, gy, qy);
                fold(cz, gz, qz);
                qx = qy = qz = 0.f;
                if (STERIC && __any(rmin < __builtin_bit_cast(unsigned, d.list_r2))) {
                    for (int u = 0; u < W; ++u) {
                        const int at = ((u ^ (u >> 1)) & 1 ? x[1] : x[0]) + (u & ~1);
                        const float4 A = sA[b][at], B = SPLIT ? sB[b][at] : A;
#pragma unroll
                        for (int q = 0; q < IPL; ++q) {
                            float rx, ry, rz;
                            if (separation(q, A, B, rx, ry, rz) < d.list_r2) {
                                const int j = c * 64 + row * 16 + (at & 15);
                                /* lanes and entries past the end stand far off, but not
                                 * out of reach where lengths are near 1e15 */
                                if (ib + q >= N || j >= N) continue;
                                append(d.nbr_cnt, d.nbr_idx, &d.ctl->flag, ib + q, j);
                                append(d.nbr_cnt, d.nbr_idx, &d.ctl->flag, j, ib + q);
                            }
                        }
                    }
                }
            }
            /* the sphere of the chunk whose sums the lane ended with */
            const int o = ((l + 48) & 48) | ((l + 14) & 15);
            float(*r)[64] = red[b][w];
            r[0][o] = cx; r[1][o] = gx; r[2][o] = cy; r[3][o] = gy; r[4][o] = cz; r[5][o] = gz;
        }
#pragma unroll
        for (int q = 0; q < IPL; ++q) {
            fold(ax[q], bx[q], px[q]);
            fold(ay[q], by[q], py[q]);
            fold(az[q], bz[q], pz[q]);
            px[q] = py[q] = pz[q] = 0.f;
        }
        if (k + 1 < it.nj) put(1 - b);
        __syncthreads();
        if (!own && t < 192) {
            const int a = t >> 6, j = c * 64 + l, J = j / BS;
            double s = 0.0;
#pragma unroll
            for (int v = 0; v < NW; ++v) s = s + ((double)red[b][v][2 * a][l] + (double)red[b][v][2 * a + 1][l]);
            if (j < N) d.part[d.sym_base[J] + ((long long)(it.i0 / BS) * 3 + a) * BS + (j - J * BS)] = s;
        }
    }
    double* out = d.part + d.sym_base[it.i0 / BS] + (long long)it.c * 3 * BS + (ib - it.i0);
#pragma unroll
    for (int q = 0; q < IPL; ++q) {
        if (ib + q < N) {
            out[q] = (double)ax[q] + (double)bx[q];
            out[BS + q] = (double)ay[q] + (double)by[q];
            out[2 * BS + q] = (double)az[q] + (double)bz[q];
        }
    }
}

template <int NW, int SPLIT>
static hipError_t go_sym(const Dev& d, const Epi& e, const Shape& sh, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    auto kern = sh.steric ? (sh.rpy ? k_pairs_sym<NW, SPLIT, 1, 1> : k_pairs_sym<NW, SPLIT, 1, 0>)
                          : (sh.rpy ? k_pairs_sym<NW, SPLIT, 0, 1> : k_pairs_sym<NW, SPLIT, 0, 0>);
    if (ev0)
        hipExtLaunchKernelGGL(kern, dim3(d.nsym), dim3(64 * NW), 0, s, ev0, ev1, 0, d, e);
    else
        hipLaunchKernelGGL(kern, dim3(d.nsym), dim3(64 * NW), 0, s, d, e);
    return hipGetLastError();
}

hipError_t launch_pairs_sym(const Dev& d, const Epi& e, const Shape& sh, hipStream_t s, hipEvent_t ev0,
                            hipEvent_t ev1) {
    if (d.nsym <= 0 || e.prec != PREC_FP32C || d.nsys != 1 || (sh.steric && !d.nbr_cnt)) return hipErrorInvalidValue;
    if (d.sym_bs == 128 * 4) return sh.split ? go_sym<4, 1>(d, e, sh, s, ev0, ev1) : go_sym<4, 0>(d, e, sh, s, ev0, ev1);
    if (d.sym_bs == 128 * 8) return sh.split ? go_sym<8, 1>(d, e, sh, s, ev0, ev1) : go_sym<8, 0>(d, e, sh, s, ev0, ev1);
    return hipErrorInvalidValue;
}

}  // namespace ad
