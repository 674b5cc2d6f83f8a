// Device helpers shared by the stencil-family kernels: deterministic block
// reductions (wavefront shuffles or DPP moves, then a fixed-order sum over the waves), the
// per-column reduction of partial sums, and the FP64 -> BF16 rounding of the
// mixed-precision Gram operands.
#pragma once
#include "qo_internal.h"

namespace qo {
namespace dev {

// Sum of v over the 64 lanes of a wavefront, complete in lane 63, by DPP moves (no LDS
// traffic, no address registers): pairs and quads by quad permutations, rows of 16 by
// row shifts, then the row sums carried up by the row broadcasts of 15 and 31.  A lane
// a move has no source for adds 0.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_sum_lane63(float v) {
    v += dpp_move<0xb1>(v);          // quad_perm [1,0,3,2]
    v += dpp_move<0x4e>(v);          // quad_perm [2,3,0,1]
    v += dpp_move<0x114>(v);         // row_shr:4
    v += dpp_move<0x118>(v);         // row_shr:8
    v += dpp_move<0x142, 0xa>(v);    // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);    // row_bcast:31 into rows 2 and 3
    return v;
}

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_move_d(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum_lane63(double v) {
    v += dpp_move_d<0xb1>(v);
    v += dpp_move_d<0x4e>(v);
    v += dpp_move_d<0x114>(v);
    v += dpp_move_d<0x118>(v);
    v += dpp_move_d<0x142, 0xa>(v);
    v += dpp_move_d<0x143, 0xc>(v);
    return v;
}

struct Red {
    double v[4][kThreads / 64];
};

template <int NQ>
__device__ __forceinline__ void block_sums(double (&v)[NQ], Red &red) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = wave_sum_lane63(v[q]);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < NQ; ++q) red.v[q][wid] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) s += red.v[q][w];
        v[q] = s;
    }
}

// Sum of part[c*tiles + t] over t, identical in every thread and every block.
__device__ __forceinline__ double col_sum(const double *__restrict__ part, int c, int tiles,
                                          Red &red) {
    double s[1] = {0.0};
    for (int t = threadIdx.x; t < tiles; t += kThreads) s[0] += part[(long)c * tiles + t];
    block_sums<1>(s, red);
    return s[0];
}

// col_sum in three steps, for a workgroup of 128 or of 256 and more threads that has other
// work between them: the loads of a column's partials, the wavefronts' sums into red[4],
// and, after a barrier, the total.  Same order of additions as col_sum, so the same bits.
struct ColParts {
    double a, b;  // this thread's terms: as thread tid and, of 128 threads, as thread 128 + tid
};
__device__ __forceinline__ ColParts col_parts(const double *__restrict__ part, int tiles) {
    auto terms = [&](int t) {
        double s = 0.0;
        if (t < tiles) {
            s = part[t];
            for (t += kThreads; t < tiles; t += kThreads) s += part[t];
        }
        return s;
    };
    const int tid = threadIdx.x;
    return {tid < kThreads ? terms(tid) : 0.0, blockDim.x < kThreads ? terms(tid + 128) : 0.0};
}
__device__ __forceinline__ void col_parts_put(ColParts v, double *red) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    v.a = wave_sum_lane63(v.a);
    if (lane == 63 && w < 4) red[w] = v.a;
    if (blockDim.x < kThreads) {
        v.b = wave_sum_lane63(v.b);
        if (lane == 63) red[w + 2] = v.b;
    }
}
__device__ __forceinline__ double col_parts_get(const double *red) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += red[w];
    return s;
}

// Sum of lanes 0..15, in every lane (the other lanes' values do not count).
__device__ __forceinline__ double row_sum16(double v) {
    v += dpp_move_d<0xb1>(v);
    v += dpp_move_d<0x4e>(v);
    v += dpp_move_d<0x114>(v);
    v += dpp_move_d<0x118>(v);
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, 15);
    const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 15);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Several such sums at once: v[q] = sum of p[q][0 .. n[q] - 1].  Their loads are under way
// together and they share one reduction.
template <int NQ>
__device__ __forceinline__ void part_sums(const double *const (&p)[NQ], const int (&n)[NQ],
                                          double (&v)[NQ], Red &red) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        v[q] = 0.0;
        for (int t = threadIdx.x; t < n[q]; t += kThreads) v[q] += p[q][t];
    }
    block_sums<NQ>(v, red);
}

// Round an FP64 value to bfloat16, nearest-even on the 45 dropped mantissa bits (one
// rounding, no FP32 intermediate).  Magnitudes below the FP32 normal range flush to signed
// zero; beyond it saturate to infinity; NaN becomes the quiet NaN.  Straight-line form: the
// rounded magnitude's bits 45..59 are the exponent and the 7 kept mantissa bits, rebiased
// to BF16 with selects instead of branches.
__device__ __forceinline__ __bf16 f64_to_bf16_rne(double d) {
    const unsigned long long b = __double_as_longlong(d);
    const unsigned long long mag =
        (b & 0x7fffffffffffffffull) + 0xfffffffffffull + ((b >> 45) & 1ull);
    int v = (int)(unsigned int)(mag >> 45) - ((1023 - 127) << 7);
    v = v < 0x80 ? 0 : v;
    v = min(v, 0x7f80);
    v = __builtin_isnan(d) ? 0x7fc0 : v;
    const unsigned int s16 = (unsigned int)(b >> 48) & 0x8000u;
    return __builtin_bit_cast(__bf16, (unsigned short)(s16 | (unsigned int)v));
}

}  // namespace dev
}  // namespace qo
