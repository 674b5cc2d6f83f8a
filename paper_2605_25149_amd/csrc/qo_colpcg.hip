// FP64 Jacobi-PCG that keeps its columns on the chip: the inverse operator
// G = H_sigma^{-1} of Sec. 3.1 with a whole column per workgroup (k_pcg_column, grids of at most
// kColPcgMax = 16384 points) or per cluster of up to kCluMaxW = 64 workgroups of at most
// kCluPts = 8192 points each (k_pcg_cluster, up to 524288 points; second part of this file).
//
// The streaming form (qo_stencil.hip) takes two launches per iteration, each a chain of
// flag loads, partial-sum reductions and plane passes of 5 to 6 us however small the grid;
// a 32 x 32 solve of some 120 iterations then costs 1.9 ms.
//
// A workgroup per column: it keeps its column on the CU for the whole solve, x, r and the
// search direction in registers, a copy of the direction in LDS for the neighbours, and
// the dot products as wavefront sums exchanged through LDS.  An iteration is three barriers
// and touches no global memory (above 8 points per thread x and the per-point arrays V + sigma
// and 1/diag stay in L2, and the thread's own direction is read back from LDS).  Columns are
// independent, so a solve of N columns is one launch of N workgroups.
//
// A cluster per column exchanges faces, partial sums and counters through global memory every
// iteration and needs its workgroups on the chip together; what that takes stands with it.
//
// Bound of the first form: latency of the two reductions on the smallest grids, LDS traffic
// (five accesses per point in 2-D, seven in 3-D) and the FP64 rate of the column's CU on the
// larger ones, the L2 round trips above 8192 points.  Measured times stand at the launch.
//
// Both: same iteration, stop test and error conditions as the streaming form; the dot products
// are summed in another order.
#include "qo_device.h"
#include "qo_internal.h"

#include <algorithm>
#include <mutex>

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

// ---- a column per cluster of workgroups
//
// Grids of more than kCluPts points: W workgroups share a column, each with a box of at most
// kCluPts points (whole rows along x, a range of y and z; in 2-D a range of rows) held as in
// k_pcg_column (16 per thread, in registers but for the direction) and, in LDS, the
// direction over the box and one layer around it.  Two exchanges per iteration, each a partial
// sum per workgroup and a counter that every workgroup of the cluster waits on: gamma, and
// then r.z with ||r||^2, before which the preconditioned residual z = D r on the box's faces is
// published.  A workgroup keeps the neighbours' part of the direction itself (p = z + beta p,
// beta the same everywhere), so the direction needs no exchange of its own.  Every workgroup
// adds the same partials in the same order and so takes the same decisions.
//
// What is exchanged (faces, partials, counters) is written and read with agent-scope atomic
// accesses alone, which are coherent across the XCDs' L2 caches: a wavefront's stores have
// arrived when its wait on them ends, the workgroup's barrier and the counter come after
// that, and a reader issues its loads after it has seen the counter.  Agent-scope fences
// would write back and invalidate whole L2 caches for data that never sits there
// (64^3, 64 columns: 18.1 instead of 12.6 us an iteration).
//
// Bound: the two waits (about 5 us an iteration together), the faces' round trip, and the LDS
// traffic and FP64 rate of one CU per box.  Boxes rather than ranges of the linear index,
// because their faces are smaller (64^3 over 32 workgroups: 3072 values each instead of 8192).
// Whole solves, tol 1e-10, against the streaming sweeps: 64^3 x 64 columns 89.9 -> 34.6 ms
// (eight columns at a time), 70 x 70 x 80 x 64 163 -> 65 ms, 40^3 x 64 24.0 -> 4.9 ms, 199^2 x
// 64 48.4 -> 12.3 ms, 256^2 x 256 332 -> 62.9 ms, 64^3 x 4 21.3 -> 4.1 ms.
//
// All workgroups of a launch have to be resident at once.  Within a process they are: there are
// at most as many as CUs, each CU holds at least one, other kernels end by themselves, and
// two such launches never meet on a device (each waits for the event of the one before it).
// Another process on the GPU, or a kernel that itself waits for something, can hold CUs for
// longer.  So every wait is bounded: a workgroup that runs out of polls raises `abort`, on
// which all of them leave, and the host takes another form for the rest of the handle's life.
// A cooperative launch would ensure no more, and after the first one of a process its streams
// overlap less: 16 grouped problems on four streams stepped in 86 ms instead of 70 from then
// on.
constexpr int kCluThreads = 512;
constexpr int kCluPts = 8192;      // 512 threads x 16 (1024 x 8 spills some 80 registers)
constexpr int kCluMaxW = 64;       // one partial per lane of a wavefront
constexpr int kCluPolls = 1 << 21; // a poll is about half a microsecond
constexpr int kCluCtr = 16;        // ints between two counters
constexpr int kCluDevices = 64;    // devices a process may use

__device__ __forceinline__ void pub(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double obs(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// This wavefront's published values have arrived, and no store before is moved behind: the
// wait alone touches no memory in the compiler's model, and a relaxed store could sink below.
__device__ __forceinline__ void published() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
}

struct CluSync {
    int *abort, *ctr;    // this cluster's counter
    double *slots;       // [2][3][kCluMaxW]: parity, value, workgroup
    int W, w, epoch;
};

// v summed over the cluster, the same bits in every thread of it; everything published
// before is visible after it.  False: the wait ran out (uniform over the workgroup).
template <int NQ>
__device__ __forceinline__ bool clu_sums(double (&v)[NQ], CluSync &c, double (*sh)[16],
                                         double *res) {
    static_assert(NQ <= 3, "three slots per workgroup and parity");
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dev::wave_sum_lane63(v[q]);
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < NQ; ++q) sh[q][wid] = v[q];
    published();
    __syncthreads();
    if (wid == 0) {
        ++c.epoch;
        double *slot = c.slots + (c.epoch & 1) * 3 * kCluMaxW;
        double t[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) t[q] = dev::row_sum16(lane < nw ? sh[q][lane] : 0.0);
        int ok = 1;
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) pub(slot + q * kCluMaxW + c.w, t[q]);
            published();
            __hip_atomic_fetch_add(c.ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int target = c.epoch * c.W;
            int n = 0;
            while (__hip_atomic_load(c.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if (++n >= kCluPolls ||
                    ((n & 1023) == 0 &&
                     __hip_atomic_load(c.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    __hip_atomic_store(c.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = 0;
                    break;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
        ok = __builtin_amdgcn_readfirstlane(ok);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double x = lane < c.W ? obs(slot + q * kCluMaxW + lane) : 0.0;
            const double s = dev::wave_sum_lane63(x);
            if (lane == 63) res[q] = s;
        }
        if (lane == 63) res[3] = ok ? 0.0 : 1.0;
    } else {
        ++c.epoch;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = res[q];
    return res[3] == 0.0;
}

struct CluShape {
    int W, Wy, Wz;  // workgroups per column (0: another path), along y and z
    int by, bz;     // rows and planes of a box (2-D: by = 1, bz rows)
    size_t smem;
};

// Iterations k0 .. kend for the columns c0 .. c1 - 1; otherwise as k_pcg_column.  Zx: the
// published z; Rw, Pw: r and p of columns to be continued.
template <bool D3>
__global__ __launch_bounds__(kCluThreads) void k_pcg_cluster(
    Grid g, const double *__restrict__ vs, const double *__restrict__ dinv,
    const double *__restrict__ B, double *__restrict__ X, double *Zx, double *__restrict__ Rw,
    double *__restrict__ Pw, long ld, int use_x0, double tol, int k0, int kend, bool last,
    double *__restrict__ scal, int *__restrict__ its, int *__restrict__ state, CluShape sh, int c0,
    int c1, int *ctl, double *slots) {
    constexpr int NT = kCluThreads, PPT = kCluPts / NT;
    extern __shared__ double P[];  // the box with one layer of planes (and, in 3-D, rows) around
    __shared__ double red[2][3][16], res[2][4];
    const int tid = threadIdx.x;
    const int W = sh.W, nclus = (int)gridDim.x / W;
    const int L = xcd_remap(blockIdx.x, gridDim.x);  // a cluster's workgroups on one XCD
    const int clu = L / W, w = L - clu * W;
    CluSync cs{ctl, ctl + kCluCtr * (1 + clu), slots + (size_t)clu * 6 * kCluMaxW, W, w, 0};
    // the grid as nx x NY x NZ (2-D: NY = 1), the box [y0, y0 + ly) x [z0, z0 + lz)
    const int nx = g.nx, NY = D3 ? g.ny : 1, NZ = D3 ? g.nz : g.ny;
    const int y0 = (w % sh.Wy) * sh.by, z0 = (w / sh.Wy) * sh.bz;
    const int ly = min(sh.by, NY - y0), lz = min(sh.bz, NZ - z0);
    const int rowp = nx * ly, len = rowp * lz, t0 = (z0 * NY + y0) * nx;
    const int skip = nx * (NY - ly);                    // between the box's planes
    const int ps = D3 ? (ly + 2) * nx : nx, ptot = ps * (lz + 2);
    const double kap = g.kappa, cd = g.c0, ihx2 = g.ihx2, ihy2 = D3 ? g.ihy2 : 0.0,
                 ihz2 = D3 ? g.ihz2 : g.ihy2;
    // per point: LDS index (15 bits), neighbours inside the row (2), on a face that another
    // workgroup reads (1), plane of the box (13)
    unsigned pk[PPT];
    double v[PPT], d[PPT];
#pragma unroll
    for (int s = 0; s < PPT; ++s) {
        const int j = min(tid + s * NT, len - 1);
        const int z = j / rowp, q = j - z * rowp, y = q / nx, ix = q - y * nx;
        const bool face = (z == 0 && z0 > 0) || (z == lz - 1 && z0 + lz < NZ) ||
                          (y == 0 && y0 > 0) || (y == ly - 1 && y0 + ly < NY);
        pk[s] = (unsigned)((z + 1) * ps + (D3 ? nx : 0) + q) | (ix > 0 ? 1u << 15 : 0u) |
                (ix < nx - 1 ? 1u << 16 : 0u) | (face ? 1u << 17 : 0u) | (unsigned)z << 18;
        const int t = t0 + j + z * skip;
        v[s] = vs[t];
        d[s] = dinv[t];
    }
    // Addresses and tests are formed anew from values the compiler does not know: hoisted out
    // of the iteration they spill over a hundred registers.
    int tb = tid;
    auto opaque = [&] {
        asm volatile("" : "+v"(tb));
#pragma unroll
        for (int s = 0; s < PPT; ++s) asm volatile("" : "+v"(pk[s]));
    };
    auto mine = [&](int s) { return tb + s * NT < len; };
    auto li = [&](int s) { return (int)(pk[s] & 0x7fffu); };
    auto gt = [&](int s) {  // grid index (a point past the box's end: its last one)
        return (unsigned)(t0 + min(tb + s * NT, len - 1) + (int)(pk[s] >> 18) * skip);
    };
    auto apply = [&](int s, double u) {
        const int i = li(s);
        const double xm = (pk[s] & 1u << 15) ? P[i - 1] : 0.0;
        const double xp = (pk[s] & 1u << 16) ? P[i + 1] : 0.0;
        double f = ihx2 * (xm + xp);
        if constexpr (D3) f += ihy2 * (P[i - nx] + P[i + nx]);
        f += ihz2 * (P[i - ps] + P[i + ps]);
        return (cd + v[s]) * u - kap * f;
    };
    // points of the layer around the box: LDS index (-1: outside the grid, or past the last
    // one) and grid index of the i-th
    const int hy = D3 ? nx * lz : 0, nhalo = 2 * (hy + rowp);
    auto layer = [&](int i, unsigned &t) {
        if (i < 2 * hy) {
            const bool hi = i >= hy;
            const int q = hi ? i - hy : i, z = q / nx, ix = q - z * nx, y = hi ? ly : -1;
            t = (unsigned)(t0 + (z * NY + y) * nx + ix);
            return (hi ? y0 + ly >= NY : y0 == 0) ? -1 : (z + 1) * ps + (y + 1) * nx + ix;
        }
        const int i2 = i - 2 * hy;
        const bool hi = i2 >= rowp;
        const int q = hi ? i2 - rowp : i2, z = hi ? lz : -1;
        t = (unsigned)(t0 + z * NY * nx + q);
        return i >= nhalo || (hi ? z0 + lz >= NZ : z0 == 0) ? -1
                                                            : (z + 1) * ps + (D3 ? nx : 0) + q;
    };
    // P there = f(grid index)
    auto halo = [&](auto f) {
        for (int i = tb; i < nhalo; i += NT) {
            unsigned t;
            const int l = layer(i, t);
            if (l >= 0) P[l] = f(t);
        }
    };
    for (int col = c0 + clu; col < c1; col += nclus) {
        if (k0 > 0 && state[col] != kColRunning) continue;  // settled by an earlier launch
        const long o = (long)col * ld;
        double *const zx = Zx + o, *const xg = X + o, *const rg = Rw + o, *const pg = Pw + o;
        const double *const bg = B + o;
        double x[PPT], r[PPT];
        __syncthreads();  // the previous column's reads of P
        for (int i = tb; i < ptot; i += NT) P[i] = 0.0;
        __syncthreads();
        auto publish = [&](int s) {
            if (pk[s] & 1u << 17) pub(zx + gt(s), d[s] * r[s]);
        };
        double rz, rr, bb, rho_old = 0.0;
        if (k0 == 0) {
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                x[s] = use_x0 ? xg[gt(s)] : 0.0;
                r[s] = bg[gt(s)];
                if (use_x0 && mine(s)) P[li(s)] = x[s];
            }
            if (use_x0) halo([&](unsigned t) { return xg[t]; });
            __syncthreads();
            opaque();
            double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                if (!mine(s)) continue;
                const double bi = r[s];
                if (use_x0) r[s] = bi - apply(s, x[s]);
                acc[0] += r[s] * (d[s] * r[s]);
                acc[1] += r[s] * r[s];
                acc[2] += bi * bi;
                publish(s);
            }
            if (!clu_sums<3>(acc, cs, red[1], res[1])) return;
            rz = acc[0];
            rr = acc[1];
            bb = acc[2];
        } else {
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                x[s] = xg[gt(s)];
                r[s] = rg[gt(s)];
                if (mine(s)) P[li(s)] = pg[gt(s)];
            }
            halo([&](unsigned t) { return pg[t]; });
            rz = scal[4 * col];
            rr = scal[4 * col + 1];
            bb = scal[4 * col + 2];
            rho_old = scal[4 * col + 3];
        }
        int st = kColRunning, k = k0;
        for (;; ++k) {
            if (!isfinite(rz) || !isfinite(rr) || !isfinite(bb)) st = 7;
            else if (sqrt(rr) <= tol * sqrt(bb)) st = kColDone;
            if (st != kColRunning || k == kend) break;
            opaque();
            const double beta = k == 0 ? 0.0 : rz / rho_old;
            const bool first = k == 0;
            // p = z + beta p, in the layer from the neighbours' z: its first kHalo values per
            // thread are under way together (one by one, each waited out a memory round
            // trip: 19.8 us an iteration at 64^3) while the box's own are formed
            constexpr int kHalo = 8;
            double hz[kHalo];
            int hl[kHalo];
#pragma unroll
            for (int u = 0; u < kHalo; ++u) {
                unsigned t;
                hl[u] = tb + u * NT < nhalo ? layer(tb + u * NT, t) : -1;
                hz[u] = obs(zx + (hl[u] >= 0 ? t : (unsigned)t0));
            }
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                const double z = d[s] * r[s];
                if (mine(s)) P[li(s)] = first ? z : z + beta * P[li(s)];
            }
#pragma unroll
            for (int u = 0; u < kHalo; ++u)
                if (hl[u] >= 0) P[hl[u]] = first ? hz[u] : hz[u] + beta * P[hl[u]];
            for (int i = tb + kHalo * NT; i < nhalo; i += NT) {
                unsigned t;
                const int l = layer(i, t);
                if (l < 0) continue;
                const double z = obs(zx + t);
                P[l] = first ? z : z + beta * P[l];
            }
            __syncthreads();
            opaque();
            double q[PPT], gam[1] = {0.0};
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                q[s] = 0.0;
                if (!mine(s)) continue;
                const double u = P[li(s)];
                q[s] = apply(s, u);
                gam[0] += u * q[s];
            }
            if (!clu_sums<1>(gam, cs, red[0], res[0])) return;
            if (!isfinite(gam[0])) st = 7;
            else if (!(gam[0] > 0.0)) st = 5;
            if (st != kColRunning) break;
            const double alpha = rz / gam[0];
            double acc[2] = {0.0, 0.0};
            opaque();
#pragma unroll
            for (int s = 0; s < PPT; ++s) {
                if (!mine(s)) continue;
                x[s] += alpha * P[li(s)];
                r[s] -= alpha * q[s];
                acc[0] += r[s] * (d[s] * r[s]);
                acc[1] += r[s] * r[s];
                publish(s);
            }
            if (!clu_sums<2>(acc, cs, red[1], res[1])) return;
            rho_old = rz;
            rz = acc[0];
            rr = acc[1];
        }
        const bool resume = st == kColRunning && !last;
        opaque();
#pragma unroll
        for (int s = 0; s < PPT; ++s) {
            if (!mine(s)) continue;
            xg[gt(s)] = x[s];
            if (resume) {
                rg[gt(s)] = r[s];
                pg[gt(s)] = P[li(s)];
            }
        }
        if (w == 0 && tid == 0) {
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
}

size_t col_lds(const Grid &g) {
    const long pad = g.dim == 3 ? (long)g.nx * g.ny : g.nx;
    return (size_t)(g.ng + 2 * pad) * sizeof(double);
}

constexpr size_t kColLdsMax = 156 << 10;  // of the CU's 160 KiB, beside the reduction slots

}  // namespace

bool pcg_column_fits(const Grid &g) { return g.ng <= kColPcgMax && col_lds(g) <= kColLdsMax; }

// The fewest workgroups whose boxes fit the registers and the LDS, and among those the
// boxes with the smallest faces.
static CluShape clu_shape(const Grid &g) {
    CluShape best{};
    const int NY = g.dim == 3 ? g.ny : 1, NZ = g.dim == 3 ? g.nz : g.ny;
    if (g.nx > kCluPts) return best;
    long face = 0;
    for (int W = (int)std::min<long>(kCluMaxW + 1, (g.ng + kCluPts - 1) / kCluPts);
         W <= kCluMaxW && best.W == 0; ++W)
        for (int Wy = 1; Wy <= std::min(W, NY); ++Wy) {
            if (W % Wy || W / Wy > NZ) continue;
            CluShape c{W, Wy, W / Wy, (NY + Wy - 1) / Wy, 0, 0};
            c.bz = (NZ + c.Wz - 1) / c.Wz;
            // every workgroup has a box
            if ((Wy - 1) * c.by >= NY || (c.Wz - 1) * c.bz >= NZ) continue;
            const long ps = (long)g.nx * (g.dim == 3 ? c.by + 2 : 1), lds = ps * (c.bz + 2);
            c.smem = (size_t)lds * sizeof(double);
            if ((long)g.nx * c.by * c.bz > kCluPts || c.smem > kColLdsMax || lds > 0x7fff) continue;
            const long f = (long)c.by * (c.Wz > 1) + (long)c.bz * (Wy > 1);
            if (best.W == 0 || f < face) {
                best = c;
                face = f;
            }
        }
    return best;
}

int pcg_cluster_width(const Grid &g) { return clu_shape(g).W; }

size_t pcg_cluster_ints() { return kCluCtr * (1 + kCluMaxClusters); }
size_t pcg_cluster_slots() { return (size_t)6 * kCluMaxW * kCluMaxClusters; }

int pcg_cluster_count(const Grid &g) {
    int dev = 0, cus = 0, per_cu = 0;
    const CluShape sh = clu_shape(g);
    if (sh.W == 0 || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    const hipError_t e =
        g.dim == 3 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pcg_cluster<true>,
                                                                  kCluThreads, sh.smem)
                   : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pcg_cluster<false>,
                                                                  kCluThreads, sh.smem);
    if (e != hipSuccess || per_cu < 1) return 0;
    return std::min(kCluMaxClusters, cus / sh.W);  // one workgroup per CU
}

hipError_t launch_pcg_cluster(const Grid &g, int nclus, const double *vs, const double *dinv,
                              const double *B, double *X, double *Zx, double *R, double *P, long ld,
                              int c0, int c1, int use_x0, double tol, int k0, int kend, bool last,
                              double *scal, int *its, int *state, int *ctl, double *slots,
                              bool give_up, hipStream_t st) {
    if (c1 <= c0) return hipSuccess;
    CluShape sh = clu_shape(g);
    if (sh.W == 0 || g.cinst || nclus < 1 || nclus > kCluMaxClusters) return hipErrorInvalidValue;
    nclus = std::min(nclus, c1 - c0);
    // give_up: counters that no wait sees completed, and the abort flag raised
    hipError_t e = launch_fill_int(ctl, (int)pcg_cluster_ints(), give_up ? -(1 << 30) : 0, st);
    if (e != hipSuccess) return e;
    // one at a time per device (see above): each launch waits for the one before it, on
    // whichever stream and handle that was
    static std::mutex gate;
    static hipEvent_t last_done[kCluDevices] = {};
    int dev = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if (dev < 0 || dev >= kCluDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(gate);
    hipEvent_t &done = last_done[dev];
    if (!done)
        e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
    else
        e = hipStreamWaitEvent(st, done, 0);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(nclus * sh.W)), block(kCluThreads);
    if (g.dim == 3)
        hipLaunchKernelGGL(k_pcg_cluster<true>, grid, block, sh.smem, st, g, vs, dinv, B, X, Zx, R, P,
                           ld, use_x0, tol, k0, kend, last, scal, its, state, sh, c0, c1, ctl, slots);
    else
        hipLaunchKernelGGL(k_pcg_cluster<false>, grid, block, sh.smem, st, g, vs, dinv, B, X, Zx, R, P,
                           ld, use_x0, tol, k0, kend, last, scal, its, state, sh, c0, c1, ctl, slots);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return hipEventRecord(done, st);
}

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
