// Gauss-Jordan solve B <- A^{-1} B of a small system by one workgroup, matrix in registers.
#pragma once
#include "qo_device.h"

namespace qo {
namespace dev {

constexpr int kGjRegWaves = 16;             // wavefronts of the workgroup
constexpr int kGjRegN = 64;                 // rows: one per lane
constexpr int kGjRegCols = 8 * kGjRegWaves; // columns of [A | B]

struct GjShared {
    double f[2][64];  // the pivot column of the even / odd steps
    double inv[2];
    int p[2], fail[2];
};

__device__ __forceinline__ double read_lane(double v, int lane) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Maximum of non-negative values over the wavefront, in every lane: the moves of
// wave_sum_lane63 (a missing source is 0), then lane 63.  By LDS permutes a 32 x 32
// solve took 23.7 us, so 22.0.
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_move_d<0xb1>(v));
    v = fmax(v, dpp_move_d<0x4e>(v));
    v = fmax(v, dpp_move_d<0x114>(v));
    v = fmax(v, dpp_move_d<0x118>(v));
    v = fmax(v, dpp_move_d<0x142, 0xa>(v));
    v = fmax(v, dpp_move_d<0x143, 0xc>(v));
    return read_lane(v, 63);
}

// n <= 64, n + m <= 16 CPW, 1024 threads.  spd: no pivoting, fail (5) when a pivot is not above
// 1e-13 of the largest diagonal entry; else partial pivoting.  Returns the status (0 ok, 5
// singular / not SPD, 7 non-finite; B is then unchanged), identical in every thread.  A is
// not changed.
//
// Lane i holds row i of columns w, w + 16, ... of [A | B] for wavefront w.  A step costs one
// barrier: the wavefront of column k + 1 takes it through step k first, chooses its pivot
// and publishes it (column, reciprocal, row) in the other half of sh, while the rest of the
// columns follow.  Rows are not swapped: a row that has been the pivot of step k is marked,
// and holds row k of the solution in the end.  With the matrix in global memory and six
// barriers per step the two solves of a step took about 130 us for 32 columns (44 now).
template <int CPW>
__device__ __forceinline__ int gj_reg(const double *A, int lda, double *B, int ldb, int n, int m,
                                      bool spd, GjShared &sh) {
    constexpr int NW = kGjRegWaves;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    double x[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        const int j = w + NW * c;
        x[c] = 0.0;
        if (lane < n && j < n + m)
            x[c] = j < n ? A[(long)j * lda + lane] : B[(long)(j - n) * ldb + lane];
    }
    double thr = 0.0;
    if (spd) thr = 1e-13 * wave_max(lane < n ? fabs(A[(long)lane * lda + lane]) : 0.0);
    bool used = lane >= n;
    int var = 0;  // the unknown that this lane's row ends up holding
    auto publish = [&](int k, double v) {
        int p = k, fail = 0;
        double pv;
        if (spd) {
            pv = read_lane(v, k);
            if (!(pv > thr) || !isfinite(pv)) fail = isfinite(pv) ? 5 : 7;
        } else {
            const double a = used || v != v ? 0.0 : fabs(v);  // a NaN is never the pivot
            const double best = wave_max(a);
            if (!(best > 0.0) || !isfinite(best)) fail = isfinite(best) ? 5 : 7;
            const unsigned long long at = __ballot(!used && a == best);
            p = at ? __ffsll(at) - 1 : 0;
            pv = read_lane(v, p);
        }
        sh.f[k & 1][lane] = v;
        if (lane == 0) {
            sh.inv[k & 1] = 1.0 / pv;
            sh.p[k & 1] = p;
            sh.fail[k & 1] = fail;
        }
    };
    if (w == 0) publish(0, x[0]);
    __syncthreads();
    int status = 0;
#pragma unroll
    for (int c0 = 0; c0 < CPW; ++c0) {
        for (int r = 0; r < NW; ++r) {
            const int k = c0 * NW + r;
            if (k >= n || status) break;
            const int p = __builtin_amdgcn_readfirstlane(sh.p[k & 1]);
            const double f = sh.f[k & 1][lane], inv = sh.inv[k & 1];
            status = __builtin_amdgcn_readfirstlane(sh.fail[k & 1]);
            if (status) break;
            const bool isp = lane == p;
            if (isp) {
                used = true;
                var = k;
            }
            auto step = [&](int c) {
                const double pr = read_lane(x[c], p) * inv;
                x[c] = isp ? pr : x[c] - f * pr;
            };
            const bool wrap = r == NW - 1;                 // column k + 1 is in the next slot
            const bool own = w == (wrap ? 0 : r + 1);      // ... and this wavefront's
            if (own && !wrap) {
                step(c0);
                if (k + 1 < n) publish(k + 1, x[c0]);
            } else if (w > r) {
                step(c0);
            }
            if (c0 + 1 < CPW) {
                step(c0 + 1 < CPW ? c0 + 1 : c0);
                if (own && wrap && k + 1 < n) publish(k + 1, x[c0 + 1 < CPW ? c0 + 1 : c0]);
            }
#pragma unroll
            for (int c = c0 + 2; c < CPW; ++c) step(c);
            __syncthreads();
        }
    }
    if (!status) {
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            const int j = w + NW * c;
            if (lane < n && j >= n && j < n + m) B[(long)(j - n) * ldb + var] = x[c];
        }
    }
    __syncthreads();
    return status;
}

// any n <= 64 with n + m <= 128
__device__ __forceinline__ int gj_reg(const double *A, int lda, double *B, int ldb, int n, int m,
                                      bool spd, GjShared &sh) {
    if (n + m <= kGjRegWaves) return gj_reg<1>(A, lda, B, ldb, n, m, spd, sh);
    if (n + m <= 2 * kGjRegWaves) return gj_reg<2>(A, lda, B, ldb, n, m, spd, sh);
    if (n + m <= 4 * kGjRegWaves) return gj_reg<4>(A, lda, B, ldb, n, m, spd, sh);
    return gj_reg<8>(A, lda, B, ldb, n, m, spd, sh);
}

}  // namespace dev
}  // namespace qo
