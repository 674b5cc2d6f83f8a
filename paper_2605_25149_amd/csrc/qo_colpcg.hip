// FP64 Jacobi-PCG of small grids with a whole column per workgroup: the inverse operator
// G = H_sigma^{-1} of Sec. 3.1 for grids of at most kColPcgMax points.
//
// The streaming form (qo_stencil.hip) takes two launches per iteration, each a chain of
// flag loads, partial-sum reductions and plane passes of 5 to 6 us however small the grid;
// a 32 x 32 solve of some 120 iterations then costs 1.9 ms.  Here one workgroup
// keeps its column on the CU for the whole solve: x, r and the search direction in
// registers, a copy of the direction in LDS for the neighbours, and the dot products as
// wavefront sums exchanged through LDS.  An iteration is three barriers and touches
// no global memory (above 8 points per thread x and the per-point arrays V + sigma and
// 1/diag stay in L2, and the thread's own direction is read back from LDS).
// Columns are independent, so a solve of N columns is one launch of N workgroups.
//
// Bound: latency of the two reductions on the smallest grids, LDS traffic (five accesses
// per point in 2-D, seven in 3-D) and the FP64 rate of the column's CU on the larger ones,
// the L2 round trips above 8192 points.  Measured times stand at the launch.
//
// Same iteration, stop test and error conditions as the streaming form; the dot products
// are summed in another order.
#include "qo_device.h"
#include "qo_internal.h"

namespace qo {

namespace {

// Sum over the workgroup, the same bits in every thread: wavefront sums through sh (one slot
// per wavefront and value), then every wavefront adds the slots.  One barrier; the caller
// alternates between two sets of slots.
template <int NQ>
__device__ __forceinline__ void col_sums(double (&v)[NQ], double (*sh)[16], int nw) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dev::wave_sum_lane63(v[q]);
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < NQ; ++q) sh[q][w] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dev::row_sum16(lane < nw ? sh[q][lane] : 0.0);
}

// Iterations k0 .. kend of the solve (kend < maxit: to be continued by a launch from kend).
// KEEP: x, the direction and the per-point arrays stay in registers.  D3: 3-D grid.
template <int PPT, int NT, bool KEEP, bool D3>
__global__ __launch_bounds__(NT) void k_pcg_column(Grid g, const double *__restrict__ vs,
                                                   const double *__restrict__ dinv,
                                                   const double *__restrict__ B,
                                                   double *__restrict__ X,
                                                   double *__restrict__ R,
                                                   double *__restrict__ Pw, long ld, int use_x0,
                                                   double tol, int k0, int kend, bool last,
                                                   double *__restrict__ scal,
                                                   int *__restrict__ its,
                                                   int *__restrict__ state) {
    extern __shared__ double lds[];
    __shared__ double red[2][3][16];
    const int col = blockIdx.x, tid = threadIdx.x;
    if (k0 > 0 && state[col] != kColRunning) return;  // settled by an earlier launch
    const int nx = g.nx, ny = g.ny, ng = (int)g.ng, plane = nx * ny;
    const int pad = D3 ? plane : nx;
    double *P = lds + pad;  // P[t], zeros on both sides for the rows / planes outside
    constexpr int nw = NT / 64;
    const double kap = g.kappa, c0 = g.c0, ihx2 = g.ihx2, ihy2 = g.ihy2, ihz2 = g.ihz2;
    const double *b = B + (long)col * ld;
    double *xg = X + (long)col * ld, *rg = R + (long)col * ld, *pg = Pw + (long)col * ld;

    // neighbours inside the row (bits 0, 1) and, in 3-D, inside the plane (bits 2, 3); the
    // outermost ones of the grid fall into the zero padding
    unsigned long long nbs = 0;  // four bits per point
    double x[KEEP ? PPT : 1], r[PPT], p[KEEP ? PPT : 1], v[KEEP ? PPT : 1], d[KEEP ? PPT : 1];
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int t = tid + s * NT;
        const int row = t / nx, ix = t - row * nx, iy = D3 ? row % ny : 0;
        const unsigned nb = (ix > 0 ? 1u : 0u) | (ix < nx - 1 ? 2u : 0u) | (iy > 0 ? 4u : 0u) |
                            (iy < ny - 1 ? 8u : 0u);
        nbs |= (unsigned long long)nb << (4 * s);
        const int tc = min(t, ng - 1);
        const double x0 = (use_x0 || k0 > 0) ? xg[tc] : 0.0, p0 = k0 > 0 ? pg[tc] : 0.0;
        if constexpr (KEEP) {
            v[s] = vs[tc];
            d[s] = dinv[tc];
            x[s] = x0;
            p[s] = p0;
        } else if (t < ng) {
            P[t] = k0 > 0 ? p0 : x0;
            if (!use_x0 && k0 == 0) xg[t] = 0.0;
        }
        r[s] = k0 > 0 ? rg[tc] : b[tc];
    }
    for (int i = tid; i < pad; i += NT) lds[i] = lds[pad + ng + i] = 0.0;

    // !KEEP: addresses formed anew from tb, whose value the compiler does not know to be tid,
    // in groups of four points: hoisted out of the iteration, or with the loads of all 16
    // points moved together, they spill some 140 registers.
    int tb = tid;
    auto fence = [&](int s) {
        if constexpr (!KEEP)
            if ((s & 3) == 3) {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("" : "+v"(tb));
            }
    };
    auto at = [&](const double *a, const double *kept, int s) {
        return KEEP ? kept[KEEP ? s : 0] : a[tb + s * NT];
    };
    // the thread's own value of the direction
    auto own = [&](int s) { return KEEP ? p[KEEP ? s : 0] : P[tb + s * NT]; };
    // H_sigma of the function in P at point s, u = its own value there
    auto apply = [&](int s, double u) {
        const int t = (KEEP ? tid : tb) + s * NT;
        const unsigned nb = (unsigned)(nbs >> (4 * s));
        const double xm = (nb & 1) ? P[t - 1] : 0.0, xp = (nb & 2) ? P[t + 1] : 0.0;
        double ym = P[t - nx], yp = P[t + nx];
        double zz = 0.0;
        if constexpr (D3) {
            ym = (nb & 4) ? ym : 0.0;
            yp = (nb & 8) ? yp : 0.0;
            zz = ihz2 * (P[t - plane] + P[t + plane]);
        }
        return (c0 + at(vs, v, s)) * u - kap * (ihx2 * (xm + xp) + ihy2 * (ym + yp) + zz);
    };

    double rz, rr, bb, rho_old = 0.0;
    if (k0 == 0) {
        double acc[3] = {0.0, 0.0, 0.0};
        if constexpr (KEEP)
            if (use_x0) {
#pragma unroll
                for (int s = 0; s < PPT; ++s)
                    if (tid + s * NT < ng) P[tid + s * NT] = x[s];
            }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            fence(s);
            if (tid + s * NT >= ng) continue;
            const double bi = r[s];
            if (use_x0) r[s] = bi - apply(s, KEEP ? x[KEEP ? s : 0] : P[tid + s * NT]);
            acc[0] += r[s] * (at(dinv, d, s) * r[s]);
            acc[1] += r[s] * r[s];
            acc[2] += bi * bi;
        }
        col_sums<3>(acc, red[1], nw);
        rz = acc[0];
        rr = acc[1];
        bb = acc[2];
    } else {
        rz = scal[4 * col];
        rr = scal[4 * col + 1];
        bb = scal[4 * col + 2];
        rho_old = scal[4 * col + 3];
    }
    int st = kColRunning, k = k0;
    for (;; ++k) {
        // the stop test of the first sweep
        if (!isfinite(rz) || !isfinite(rr) || !isfinite(bb)) st = 7;
        else if (sqrt(rr) <= tol * sqrt(bb)) st = kColDone;
        if (st != kColRunning || k == kend) break;
        const double beta = k == 0 ? 0.0 : rz / rho_old;
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            fence(s);
            if (!KEEP && tb + s * NT >= ng) continue;
            const double z = at(dinv, d, s) * r[s];
            const double pn = k == 0 ? z : z + beta * own(s);
            if constexpr (KEEP) p[s] = pn;
            if (!KEEP || tid + s * NT < ng) P[(KEEP ? tid : tb) + s * NT] = pn;
        }
        __syncthreads();
        double q[PPT], gam[1] = {0.0};
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            q[s] = 0.0;
            fence(s);
            if ((KEEP ? tid : tb) + s * NT >= ng) continue;
            const double u = own(s);
            q[s] = apply(s, u);
            gam[0] += u * q[s];
        }
        col_sums<1>(gam, red[0], nw);
        if (!isfinite(gam[0])) st = 7;
        else if (!(gam[0] > 0.0)) st = 5;
        if (st != kColRunning) break;
        const double alpha = rz / gam[0];
        double acc[2] = {0.0, 0.0};
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            fence(s);
            if ((KEEP ? tid : tb) + s * NT >= ng) continue;
            if constexpr (KEEP) x[s] += alpha * p[s];
            else xg[tb + s * NT] += alpha * own(s);
            r[s] -= alpha * q[s];
            acc[0] += r[s] * (at(dinv, d, s) * r[s]);
            acc[1] += r[s] * r[s];
        }
        col_sums<2>(acc, red[1], nw);
        rho_old = rz;
        rz = acc[0];
        rr = acc[1];
    }
    const bool resume = st == kColRunning && !last;
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int t = tid + s * NT;
        if (t >= ng) continue;
        if constexpr (KEEP) xg[t] = x[s];
        if (resume) {
            rg[t] = r[s];
            pg[t] = own(s);
        }
    }
    if (tid == 0) {
        its[col] = k;
        state[col] = st;
        if (resume) {
            scal[4 * col] = rz;
            scal[4 * col + 1] = rr;
            scal[4 * col + 2] = bb;
            scal[4 * col + 3] = rho_old;
        }
    }
}

size_t col_lds(const Grid &g) {
    const long pad = g.dim == 3 ? (long)g.nx * g.ny : g.nx;
    return (size_t)(g.ng + 2 * pad) * sizeof(double);
}

constexpr size_t kColLdsMax = 156 << 10;  // of the CU's 160 KiB, beside the reduction slots

}  // namespace

bool pcg_column_fits(const Grid &g) { return g.ng <= kColPcgMax && col_lds(g) <= kColLdsMax; }

hipError_t launch_pcg_column(const Grid &g, const double *vs, const double *dinv, const double *B,
                             double *X, double *R, double *P, long ld, int ncols, int use_x0,
                             double tol, int k0, int kend, bool last, double *scal, int *its,
                             int *state, hipStream_t st) {
    if (ncols <= 0) return hipSuccess;
    if (!pcg_column_fits(g) || g.cinst) return hipErrorInvalidValue;
    const size_t smem = col_lds(g);
#define QO_COL(PPT, NT, KEEP)                                                                  \
    do {                                                                                       \
        if (g.dim == 3)                                                                        \
            hipLaunchKernelGGL((k_pcg_column<PPT, NT, KEEP, true>), dim3(ncols), dim3(NT), smem, \
                               st, g, vs, dinv, B, X, R, P, ld, use_x0, tol, k0, kend, last,   \
                               scal, its, state);                                              \
        else                                                                                   \
            hipLaunchKernelGGL((k_pcg_column<PPT, NT, KEEP, false>), dim3(ncols), dim3(NT),    \
                               smem, st, g, vs, dinv, B, X, R, P, ld, use_x0, tol, k0, kend,   \
                               last, scal, its, state);                                        \
    } while (0)
    // Microseconds per iteration (N = 64; the streaming sweeps in brackets): 32^2 1.73 (15.8),
    // 45^2 1.80 (16.9), 64^2 2.17 (17.5), 90^2 3.18 (19.0), 128^2 13.2 (29.3), 16^3 2.89
    // (27.7), 20^3 4.14 (42.8), 25^3 14.3 (73.4).  Other shapes: 32^2 as 256 x 4 1.83, 128 x 8
    // 2.11, 64 x 16 2.99; 45^2 as 1024 x 2 2.43, 256 x 8 2.25; 64^2 as 1024 x 4 2.72; 90^2 as
    // 512 x 16 3.46.
    if (g.ng <= 1024) QO_COL(2, 512, true);
    else if (g.ng <= 2048) QO_COL(4, 512, true);
    else if (g.ng <= 4096) QO_COL(8, 512, true);
    else if (g.ng <= 8192) QO_COL(8, 1024, true);
    else QO_COL(16, 1024, false);
#undef QO_COL
    return hipGetLastError();
}

}  // namespace qo
