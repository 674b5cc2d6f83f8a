// Tall-skinny Gram matrices <Z,Z> = w Z^T Z of Z = [X | Y] (Ng x 2n): the
// inner-product matrices of Sec. 2.1 that the scheme of Sec. 4.1 needs
// (<U,U>, <U,GU>, <GU,GU> and <U_hat,U_hat>, <U_hat,GU_hat>, <GU_hat,GU_hat>).
//
// Split-K over the grid: a workgroup computes one 64x64 tile of the upper
// block triangle over one chunk of rows with MFMA (FP64: four wavefronts, a
// quarter of the rows each, summed through LDS), writes it as a partial, and a
// second kernel sums the partials of every entry in a fixed order and mirrors
// the upper triangle (deterministic, exactly symmetric).
//
// Operand trick: the sum over grid rows may visit the rows in any order as
// long as both operands use the same order, so lane l takes rows
// k0 + R*(l/16) + s (s < R) for its MFMA slot (l/16, l%16): each lane reads R
// consecutive doubles of one column instead of a strided gather.
//   FP64: v_mfma_f64_16x16x4f64, R = 4.
//   BF16: v_mfma_f32_16x16x32_bf16, R = 8, inputs rounded to nearest-even
//         from FP64, FP32 accumulation within a chunk, FP64 across chunks.
#include "qo_internal.h"
#include "qo_device.h"

#include <algorithm>
#include <type_traits>


namespace qo {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int TM = 64;         // output tile edge per workgroup (FP64) or wavefront (BF16)
constexpr int kGramWaves = 4;  // FP64: wavefronts per workgroup, each with a part of the rows
constexpr size_t kGramLds = (size_t)kGramWaves * TM * TM * sizeof(double);

// Global-address-space views.  Pointers read from a job table are generic; generic loads
// count on both the vector-memory and the LDS/scalar counters, and the compiler then
// waits for all of them before the MFMAs, which defeats the prefetch.
typedef const double __attribute__((address_space(1))) gdouble;
typedef double d2 __attribute__((ext_vector_type(2)));
typedef const d2 __attribute__((address_space(1))) gd2;
__device__ __forceinline__ gdouble *gptr(const double *p) { return (gdouble *)p; }

__device__ __forceinline__ const double *zcol(const double *X, const double *Y, long ld, int n,
                                              int c) {
    return c < n ? X + (long)c * ld : Y + (long)(c - n) * ld;
}

using dev::f64_to_bf16_rne;

// Decode the upper-triangular tile pair index.
__device__ __forceinline__ void tile_pair(int p, int nt, int &ti, int &tj) {
    int i = 0, rem = p;
    while (rem >= nt - i) {
        rem -= nt - i;
        ++i;
    }
    ti = i;
    tj = i + rem;
}

// One wavefront's rows [kb, ke) of a tile of NI x NJ blocks of 16 x 16 (DIAG: a diagonal
// tile, whose operands coincide and whose blocks below the diagonal are left out): acc is
// left in LDS layout order, slot 4 i + j.  VEC: 16-byte aligned columns; kVecRuntime: by vec_ok,
// for the 4 x 4 form of a kernel that holds no other: its two loops then share one end, and the
// compiler leaves acc in the accumulation registers (one copy of the form for each
// alignment moved eight of them to and fro in every iteration).
enum { kVecNo, kVecYes, kVecRuntime };
template <int NI, int NJ, bool DIAG, int VEC, int W>
__device__ __forceinline__ void gram_rows(const double *const (&pa_)[4],
                                          const double *const (&pb_)[4], long kb, long ke,
                                          double *__restrict__ red, double *__restrict__ out,
                                          int wave, int nn, int r0t, int c0t, int vec_ok) {
    constexpr int NB = DIAG ? 1 : NJ;  // column groups of B loaded
    static_assert(W == 1 || W == 4, "W = 4: one value of a block per wavefront in the final sum");
    const int lr = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
    gdouble *pa[NI], *pb[NB];
#pragma unroll
    for (int i = 0; i < NI; ++i) pa[i] = gptr(pa_[i]);
#pragma unroll
    for (int j = 0; j < NB; ++j) pb[j] = gptr(pb_[j]);
    v4d acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    auto mma_chunk = [&](const double (&a)[NI][4], const double (&b)[NB][4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = DIAG ? i : 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        a[i][s], DIAG ? a[j < NI ? j : 0][s] : b[j < NB ? j : 0][s], acc[i][j], 0,
                        0, 0);
    };
    const long len = ke > kb ? ke - kb : 0;
    const long kend = kb + (len & ~15L);
    auto main_loop = [&](auto vec) {
        auto load4 = [&](gdouble *p, long r0, double (&v)[4]) {
            if constexpr (decltype(vec)::value) {
                gd2 *q = (gd2 *)(p + r0);
                const d2 v0 = q[0], v1 = q[1];
                v[0] = v0.x; v[1] = v0.y; v[2] = v1.x; v[3] = v1.y;
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) v[s] = p[r0 + s];
            }
        };
        auto load_chunk = [&](long k0, double (&a)[NI][4], double (&b)[NB][4]) {
            const long r0 = k0 + 4 * lg;
            if constexpr (VEC == kVecRuntime) {
                // one wavefront per SIMD: in turn, so that the first products wait for the
                // first few loads alone (all of a before b: 512 columns at 96^3 rows 4.50
                // instead of 4.39 ms)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    load4(pa[i], r0, a[i]);
                    load4(pb[i], r0, b[i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < NI; ++i) load4(pa[i], r0, a[i]);
                if constexpr (!DIAG)
#pragma unroll
                    for (int j = 0; j < NB; ++j) load4(pb[j], r0, b[j]);
            }
        };
        // full chunks of 16 rows, software-pipelined one chunk ahead (past the end the
        // prefetch re-reads the final chunk); the scheduling barriers keep the prefetch ahead
        // of the MFMAs it overlaps
        if (kend <= kb) return;
        double a0[NI][4], b0[NB][4], a1[NI][4], b1[NB][4];
        const long last = kend - 16;
        const long npairs = (kend - kb) >> 5;
        load_chunk(kb, a0, b0);
        for (long p = 0; p < npairs; ++p) {
            const long k0 = kb + (p << 5);
            load_chunk(k0 + 16, a1, b1);
            __builtin_amdgcn_sched_barrier(0);
            mma_chunk(a0, b0);
            __builtin_amdgcn_sched_barrier(0);
            load_chunk(min(k0 + 32, last), a0, b0);
            __builtin_amdgcn_sched_barrier(0);
            mma_chunk(a1, b1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if ((kend - kb) & 16) mma_chunk(a0, b0);
    };
    if constexpr (VEC == kVecRuntime) {
        if (vec_ok) main_loop(std::true_type{});
        else main_loop(std::false_type{});
    } else {
        main_loop(std::bool_constant<VEC == kVecYes>{});
    }
    // tail rows [kend, ke): rows past ke are zeroed (they belong to another chunk)
    if (kend < ke) {
        const long r0 = kend + 4 * lg;
        double a[NI][4], b[NB][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool in = r0 + s < ke;
            const long r = in ? r0 + s : ke - 1;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const double x = pa[i][r];
                a[i][s] = in ? x : 0.0;
            }
            if constexpr (!DIAG)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const double y = pb[j][r];
                    b[j][s] = in ? y : 0.0;
                }
        }
        mma_chunk(a, b);
    }
    // FP64 16x16 accumulator layout: value v of lane l is row l/16 + 4v, column l%16
    if constexpr (W == 1) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = DIAG ? i : 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = r0t + 16 * i + lg + 4 * v;
                    const int c = c0t + 16 * j + lr;
                    if (r < nn && c < nn) out[(long)c * nn + r] = acc[i][j][v];
                }
        return;
    }
    // Sum over the wavefronts: every tile into LDS, then each thread adds the same entries of
    // the four in order.  The LDS stores go through an address the compiler cannot see to be
    // LDS (flat stores): LDS stores, or VALU additions into acc, make it keep acc in ordinary
    // registers and move all of it to and from the accumulation registers in every loop
    // iteration (512 columns: 4.68 instead of 4.32 ms).
    const int lane = threadIdx.x & 63;
    double *dst = red + wave * (TM * TM) + lane;
    asm("" : "+v"(dst));
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = DIAG ? i : 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) dst[64 * (16 * i + 4 * j + v)] = acc[i][j][v];
    __syncthreads();
    // this thread takes value v = wave of every block
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = DIAG ? i : 0; j < NJ; ++j) {
            const double *src = red + 64 * (16 * i + 4 * j + wave) + lane;
            double t = src[0];
#pragma unroll
            for (int w = 1; w < W; ++w) t += src[w * TM * TM];
            const int r = r0t + 16 * i + lg + 4 * wave;
            const int c = c0t + 16 * j + lr;
            if (r < nn && c < nn) out[(long)c * nn + r] = t;
        }
}

// One 64 x 64 tile pair of one K-chunk, FP64 MFMA, by W wavefronts.  W = 4: each takes a
// quarter of the chunk's rows and their tiles are summed through LDS in a fixed order, so a
// chunk costs one partial instead of one per wavefront (with one wavefront per chunk the
// partials of 96 columns at 64^3 rows were 75 MB written and read against 201 MB of
// operands).  W = 1 (many tile pairs): the wavefronts of a CU are different tile pairs of
// the same rows and share them in the caches (512 columns at 96^3 rows: 4.38 ms, 4.84 with
// W = 4).  16 x 16 blocks past the last column, or below the diagonal of a diagonal tile,
// are not computed (an FP64 MFMA occupies its matrix core for 64 cycles, and with 96 columns
// 27 of 48 blocks are of that kind): the tile's extent selects a form whose loops hold its
// blocks alone.  WHOLE (kGramTilesWhole tiles a side and more, W = 1): every tile is computed
// whole, in a kernel of that form alone.
// CROSS: the n x n block X^T Y alone (tile (ti, tj) = pair / ntn, pair % ntn over X
// columns x Y columns), partials n x n per split.
template <int W, bool CROSS = false, bool WHOLE = false>
__device__ __forceinline__ void gram_f64_tile(const double *__restrict__ X,
                                              const double *__restrict__ Y, long ld, long ng,
                                              int n, long kchunk, double *__restrict__ part,
                                              int vec_ok, int pair, int split,
                                              double *__restrict__ red) {
    const int nn = CROSS ? n : 2 * n;
    const int nt = (nn + TM - 1) / TM;
    int ti, tj;
    if (CROSS) {
        ti = pair / nt;
        tj = pair - ti * nt;
    } else {
        tile_pair(pair, nt, ti, tj);
    }
    // this wavefront's rows: its part of the chunk, in whole 16-row MFMA steps (the index is
    // made a scalar: a row count the compiler takes for divergent costs it the accumulation
    // registers of the loop)
    const int wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const long sub = ((kchunk + W - 1) / W + 15) / 16 * 16;
    const long kend_chunk = min(ng, (long)(split + 1) * kchunk);
    const long kb = min(kend_chunk, (long)split * kchunk + wave * sub);
    const long ke = min(kend_chunk, kb + sub);
    const int lr = threadIdx.x & 15;
    // Columns beyond 2n read column 0: their products only reach entries that are never
    // stored, so the loads need no guard.  (Guarded loads become branches, and the
    // compiler then waits for every load in flight before the MFMAs.)
    const double *pa[4], *pb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int ca = ti * TM + 16 * i + lr;
        const int cb = tj * TM + 16 * i + lr;
        if (CROSS) {
            pa[i] = X + (long)(ca < nn ? ca : 0) * ld;
            pb[i] = Y + (long)(cb < nn ? cb : 0) * ld;
        } else {
            pa[i] = ca < nn ? zcol(X, Y, ld, n, ca) : X;
            pb[i] = cb < nn ? zcol(X, Y, ld, n, cb) : X;
        }
    }
    double *out = part + (long)split * nn * nn;
    const int r0 = ti * TM, c0 = tj * TM;
    // column blocks of the tile; its row blocks are 4 off the diagonal of the symmetric
    // Gram (only the last tile is cut), unaligned operands take the whole tile
    const int nj = min(4, (nn - c0 + 15) / 16);
#define QO_GRAM(NI, NJ, D, V) gram_rows<NI, NJ, D, V, W>(pa, pb, kb, ke, red, out, wave, nn, r0, c0, vec_ok)
    if constexpr (WHOLE || (CROSS && W == 1)) {
        QO_GRAM(4, 4, false, kVecRuntime);
    } else if (!vec_ok) {
        if (!CROSS && ti == tj) QO_GRAM(4, 4, true, kVecNo);
        else QO_GRAM(4, 4, false, kVecNo);
    } else if (CROSS) {
        QO_GRAM(4, 4, false, kVecYes);
    } else if (ti == tj) {
        if (nj == 4) QO_GRAM(4, 4, true, kVecYes);
        else if (nj == 3) QO_GRAM(3, 3, true, kVecYes);
        else if (nj == 2) QO_GRAM(2, 2, true, kVecYes);
        else QO_GRAM(1, 1, true, kVecYes);
    } else {
        if (nj == 4) QO_GRAM(4, 4, false, kVecYes);
        else if (nj == 3) QO_GRAM(4, 3, false, kVecYes);
        else if (nj == 2) QO_GRAM(4, 2, false, kVecYes);
        else QO_GRAM(4, 1, false, kVecYes);
    }
#undef QO_GRAM
}

template <int W, bool WHOLE = false>
__global__ __launch_bounds__(64 * W) void k_gram_f64(const double *__restrict__ X,
                                                 const double *__restrict__ Y, long ld, long ng,
                                                 int n, long kchunk, double *__restrict__ part,
                                                 int vec_ok) {
    extern __shared__ double red[];
    // pairs of one K-chunk on one XCD: they read the same rows of the 2n columns
    const int nt = (2 * n + TM - 1) / TM;
    const int npairs = nt * (nt + 1) / 2;
    const int L = xcd_remap(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int split = L / npairs;
    gram_f64_tile<W, false, WHOLE>(X, Y, ld, ng, n, kchunk, part, vec_ok, L - split * npairs, split,
                                   red);
}

template <int W>
__global__ __launch_bounds__(64 * W) void k_gram_cross_f64(const double *__restrict__ X,
                                                       const double *__restrict__ Y, long ld,
                                                       long ng, int n, long kchunk,
                                                       double *__restrict__ part, int vec_ok) {
    extern __shared__ double red[];
    const int nt = (n + TM - 1) / TM;
    const int npairs = nt * nt;
    const int L = xcd_remap(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int split = L / npairs;
    gram_f64_tile<W, true>(X, Y, ld, ng, n, kchunk, part, vec_ok, L - split * npairs, split, red);
}

// Sum over the partials of 64 consecutive entries starting at e0: the workgroup's wavefronts
// take every kRedWaves-th partial, their sums are added in order.  Every load of a wavefront
// is independent and coalesced, so the pass costs a few memory round trips; one thread per
// entry walking all partials in turn cost one per partial (1024 partials of 96 columns:
// 110 us, 64 columns of the batch's 256^2 grids 34 us).  Complete in wavefront 0; the
// caller separates two calls with a barrier.
constexpr int kRedWaves = 16;
__device__ __forceinline__ double sum_parts(const double *__restrict__ part, long total,
                                            int nsplit, long e, double *__restrict__ sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double s = 0.0;
    if (e < total) {
#pragma unroll 8
        for (int k = w; k < nsplit; k += kRedWaves) s += part[(long)k * total + e];
    }
    if (w) sh[(w - 1) * 64 + lane] = s;
    __syncthreads();
    if (w == 0)
#pragma unroll
        for (int i = 0; i < kRedWaves - 1; ++i) s += sh[i * 64 + lane];
    return s;
}

// G = w sum_s part[s] (n x n, no mirroring)
__global__ __launch_bounds__(64 * kRedWaves) void k_gram_cross_reduce(
    const double *__restrict__ part, int n, int nsplit, double w, double *__restrict__ G) {
    __shared__ double sh[64 * (kRedWaves - 1)];
    const long total = (long)n * n;
    const long e = (long)blockIdx.x * 64 + (threadIdx.x & 63);
    const double s = sum_parts(part, total, nsplit, e, sh);
    if (threadIdx.x < 64 && e < total) G[e] = w * s;
}

// Grouped batches: job blockIdx.z, (pair, split) from blockIdx.x.
__global__ __launch_bounds__(64 * kGramWaves) void k_gram_f64_batch(const GramJob *__restrict__ jobs, long ld,
                                                       long ng, int vec_ok) {
    extern __shared__ double red[];
    const GramJob J = jobs[blockIdx.z];
    const int nt = (2 * J.n + TM - 1) / TM;
    const int npairs = nt * (nt + 1) / 2;
    if ((int)blockIdx.x >= npairs * J.nsplit) return;
    const int split = blockIdx.x / npairs;
    gram_f64_tile<kGramWaves>(J.X, J.Y, ld, ng, J.n, J.kchunk, J.part, vec_ok, blockIdx.x - split * npairs,
                  split, red);
}

// One FP64 block (n columns, leading dimension ld) rounded to BF16 in the row-blocked
// layout of the BF16 Gram operands: element (r, c) at ((r / 32) n + c) 32 + r % 32, rows
// ng..ld-1 zero.  A 32-row step of any set of consecutive columns is then one contiguous
// run (64 bytes per column), which the Gram kernel reads with 16-byte loads.  One thread
// per 8 rows of a (row block, column): four consecutive threads read a column's 256
// contiguous bytes, and consecutive threads write consecutive 16 bytes.
__global__ __launch_bounds__(256) void k_pack_bf16(const double *__restrict__ X, long ld,
                                                   long ng, int n, __bf16 *__restrict__ Zb) {
    const long total = (ld >> 5) * n * 4;
    for (long it = (long)blockIdx.x * blockDim.x + threadIdx.x; it < total;
         it += (long)gridDim.x * blockDim.x) {
        const long bc = it >> 2;  // (row block, column)
        const int q = (int)(it & 3);
        const long rb = bc / n;
        const int c = (int)(bc - rb * n);
        const long r0 = rb * 32 + 8 * q;
        const double *src = X + (long)c * ld + r0;
        v8bf o;
        if (r0 + 8 <= ng) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const double2 v = reinterpret_cast<const double2 *>(src)[h];
                o[2 * h] = f64_to_bf16_rne(v.x);
                o[2 * h + 1] = f64_to_bf16_rne(v.y);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = f64_to_bf16_rne(r0 + e < ng ? src[e] : 0.0);
        }
        reinterpret_cast<v8bf *>(Zb)[it] = o;
    }
}

// Gram tiles of [X | Y] from the row-blocked BF16 copies ZX of X and ZY of Y, 256-column
// super-tiles: one 1024-thread workgroup per (super-tile pair, K-chunk) stages each 32-row
// step of its two super-tiles (a contiguous run per copy) in LDS (each thread copies 16
// rows of one column), and its 16 waves each run the 16
// MFMAs of one 64 x 64 tile pair from LDS.  A column is fetched by the super-tile pairs it
// belongs to (2 for 2n = 512) instead of by every tile pair (8 to 9), and two steps of
// loads are in flight beyond the one in LDS.
constexpr int kSuper = 256;  // columns per super-tile

__global__ __launch_bounds__(1024) void k_gram_bf16_super(const __bf16 *__restrict__ ZX,
                                                          const __bf16 *__restrict__ ZY, long ld,
                                                          long ng, int n, long kchunk,
                                                          double *__restrict__ part) {
    // [buffer][super-tile a/b][column][32 rows]: a column's step is 64 bytes
    __shared__ __align__(16) __bf16 sm[2][2][kSuper][32];
    const int nn = 2 * n;
    const int nst = (nn + kSuper - 1) / kSuper;
    const int nsp = nst * (nst + 1) / 2;
    const int L = xcd_remap(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int split = L / nsp;
    int TI, TJ;
    tile_pair(L - split * nsp, nst, TI, TJ);
    // ZX and ZY are row-blocked (element (r, c) at ((r / 32) n + c) 32 + r % 32), rows
    // ng..ld-1 are zero and ld is a multiple of 64: whole 32-row steps
    const long kb = (long)split * kchunk;
    const long ke = min(ld, (min(ng, kb + kchunk) + 31) / 32 * 32);
    const int nsteps = ke > kb ? (int)((ke - kb) >> 5) : 0;
    const int tid = threadIdx.x;
    const bool two = TI != TJ;
    // copying: thread -> super-tile lt (the second one only off the diagonal), column lc,
    // rows 16 lh .. 16 lh + 15 of the step (two 16-byte loads)
    const int lt = tid >> 9, lc = (tid >> 1) & (kSuper - 1), lh = tid & 1;
    const bool loader = lt == 0 || two;
    typedef const v8bf __attribute__((address_space(1))) gv8bf;
    gv8bf *src;
    {
        const int c = (lt ? TJ : TI) * kSuper + lc;
        // columns past 2n read column 0: their products reach only entries never stored
        const __bf16 *col = c < n ? ZX + (long)c * 32 : c < nn ? ZY + (long)(c - n) * 32 : ZX;
        src = (gv8bf *)(col + (kb >> 5) * n * 32 + 16 * lh);
    }
    // steps past the end re-read the last one (their values are never stored)
    // one step is one row block: n 32-row column pieces further
    const long step = (long)n * 4;  // in 16-byte units
    auto gload = [&](int s, v8bf (&r)[2]) {
        const int sc = s < nsteps ? s : nsteps - 1;
        r[0] = src[step * sc];
        r[1] = src[step * sc + 1];
    };
    auto sstore = [&](int buf, const v8bf (&r)[2]) {
        if (loader) {
            *reinterpret_cast<v8bf *>(&sm[buf][lt][lc][16 * lh]) = r[0];
            *reinterpret_cast<v8bf *>(&sm[buf][lt][lc][16 * lh + 8]) = r[1];
        }
    };
    // compute: wave w -> tile pair (a, b) of the super-tile pair; on a diagonal super-tile
    // pair only a <= b is needed
    const int w = tid >> 6, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int a = w >> 2, b = w & 3;
    const int ti = TI * 4 + a, tj = TJ * 4 + b;
    const bool active = (two || a <= b) && ti * TM < nn && tj * TM < nn;
    const int sb = two ? 1 : 0;
    v4f acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int buf) {
        if (!active) return;
        v8bf fb[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            fb[j] = *reinterpret_cast<const v8bf *>(&sm[buf][sb][b * 64 + 16 * j + lr][8 * lg]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v8bf fa =
                *reinterpret_cast<const v8bf *>(&sm[buf][0][a * 64 + 16 * i + lr][8 * lg]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[j], acc[i][j], 0, 0, 0);
        }
    };
    if (nsteps > 0) {
        // step s sits in LDS buffer s & 1 while steps s + 1 (in r0 or r1) and s + 2 load
        v8bf r0[2], r1[2];
        gload(0, r0);
        sstore(0, r0);
        gload(1, r0);
        __syncthreads();
        int s = 0;
        for (; s + 2 <= nsteps; s += 2) {
            gload(s + 2, r1);
            __builtin_amdgcn_sched_barrier(0);
            mma(0);
            __builtin_amdgcn_sched_barrier(0);
            sstore(1, r0);
            __syncthreads();
            gload(s + 3, r0);
            __builtin_amdgcn_sched_barrier(0);
            mma(1);
            __builtin_amdgcn_sched_barrier(0);
            sstore(0, r1);
            __syncthreads();
        }
        if (s < nsteps) mma(0);  // odd step count: the last step sits in buffer 0
    }
    if (!active) return;
    double *out = part + (long)split * nn * nn;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = ti * TM + 16 * i + 4 * lg + v;
                const int c = tj * TM + 16 * j + lr;
                if (r < nn && c < nn) out[(long)c * nn + r] = (double)acc[i][j][v];
            }
}

// G[r][c] = w * sum_s part[s][min(r,c)][max(r,c)], 64 entries from 64 chunk on: each entry
// with r <= c is summed once and gives both G[r][c] and G[c][r].  FEW: by one wavefront, each
// entry's partials in turn (the same sum for up to kRedWaves of them).
template <bool FEW = false>
__device__ __forceinline__ void gram_reduce_chunk(const double *__restrict__ part, int nn,
                                                  int nsplit, double w, double *__restrict__ G,
                                                  long chunk, double *__restrict__ sh) {
    const long total = (long)nn * nn;
    const long e = chunk * 64 + (threadIdx.x & 63);
    const int c = (int)(e / nn), r = (int)(e - (long)c * nn);
    const bool mine = e < total && r <= c;
    double s = 0.0;
    if constexpr (FEW) {
        if (mine)
#pragma unroll 8
            for (int k = 0; k < nsplit; ++k) s += part[(long)k * total + e];
    } else {
        s = sum_parts(part, total, nsplit, mine ? e : total, sh);
    }
    if ((FEW || threadIdx.x < 64) && mine) {
        G[e] = w * s;
        G[(long)r * nn + c] = w * s;
    }
}

__global__ __launch_bounds__(64 * kRedWaves) void k_gram_reduce(const double *__restrict__ part,
                                                                int nn, int nsplit, double w,
                                                                double *__restrict__ G) {
    __shared__ double sh[64 * (kRedWaves - 1)];
    gram_reduce_chunk(part, nn, nsplit, w, G, blockIdx.x, sh);
}

__global__ __launch_bounds__(64 * kRedWaves) void k_gram_reduce_batch(
    const GramJob *__restrict__ jobs, double w) {
    __shared__ double sh[64 * (kRedWaves - 1)];
    const GramJob J = jobs[blockIdx.z];
    const int nn = 2 * J.n;
    const long chunks = ((long)nn * nn + 63) / 64;
    for (long ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
        gram_reduce_chunk(J.part, nn, J.nsplit, w, J.G, ch, sh);
        __syncthreads();  // sh is rewritten by the next chunk
    }
}

// ... with at most kFewParts partials per instance: four chunks per workgroup.
__global__ __launch_bounds__(256) void k_gram_reduce_batch_few(const GramJob *__restrict__ jobs,
                                                               double w) {
    const GramJob J = jobs[blockIdx.z];
    const int nn = 2 * J.n;
    const long chunks = ((long)nn * nn + 63) / 64;
    for (long ch = blockIdx.x * 4L + (threadIdx.x >> 6); ch < chunks; ch += 4L * gridDim.x)
        gram_reduce_chunk<true>(J.part, nn, J.nsplit, w, J.G, ch, nullptr);
}

}  // namespace

// Batches of many instances have few partials each (about 2048 workgroups are shared out over
// the group): sixteen wavefronts for one partial, 128 workgroups for every instance, cost 1000
// instances of 4 columns 137 us a reduction and 512 of 8 columns 72; a wavefront per 64
// entries, and no more workgroups than entries need, 4.9 and 4.8.
constexpr int kFewParts = 8;
hipError_t launch_gram_f64_batch(const GramJob *jobs, int njobs, int max_grid, int max_n,
                                 int max_split, long ld, long ng, double w, hipStream_t st) {
    if (njobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gram_f64_batch, dim3((unsigned)max_grid, 1, (unsigned)njobs),
                       dim3(64 * kGramWaves), kGramLds,
                       st, jobs, ld, ng, 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long chunks = (4L * max_n * max_n + 63) / 64;
    if (max_split <= kFewParts)
        hipLaunchKernelGGL(k_gram_reduce_batch_few,
                           dim3((unsigned)std::min(128L, (chunks + 3) / 4), 1, (unsigned)njobs),
                           dim3(256), 0, st, jobs, w);
    else
        hipLaunchKernelGGL(k_gram_reduce_batch,
                           dim3((unsigned)std::min(128L, chunks), 1, (unsigned)njobs),
                           dim3(64 * kRedWaves), 0, st, jobs, w);
    return hipGetLastError();
}

int gram_pairs(int n) {
    const int nt = (2 * n + TM - 1) / TM;
    return nt * (nt + 1) / 2;
}

long gram_kchunk(long ng, int nsplit) {
    long kchunk = (ng + nsplit - 1) / nsplit;
    return (kchunk + 31) / 32 * 32;
}

int gram_nsplit(long ng, int n) {
    const int nt = (2 * n + TM - 1) / TM;
    const int npairs = nt * (nt + 1) / 2;
    long ns = 4096 / npairs;
    const long maxk = (ng + 255) / 256;
    if (ns > maxk) ns = maxk;
    // keep the partial buffer under 256 MiB
    const long per = (long)4 * n * n * 8;
    const long cap = (256L << 20) / per;
    if (ns > cap) ns = cap;
    if (ns < 1) ns = 1;
    return (int)ns;
}

// Wavefronts per workgroup and row chunks of an FP64 Gram of npairs tile pairs, at most
// `most` chunks (what the partial buffer holds).  Up to kGramPairsW4 pairs (256 columns) four
// wavefronts: the partials of one each would be a large part of the traffic; at most
// kGramTarget workgroups, a multiple of the 256 CUs that hold one each so that the last
// round is not nearly empty, and at least 256 rows each (four 16-row steps per wavefront).
// More pairs: one wavefront and all the chunks, which share their operands' rows.
constexpr int kGramPairsW4 = 10;
// Tiles a side from which they are computed whole: trimmed ones would run ahead of the
// others on the same rows, which then meet in the caches less often (whole against trimmed:
// 512 columns at 96^3 rows 4.38 and 4.70 ms, 480 columns 4.26 and 4.61, 512 columns at
// 64^3 rows 1.68 and 1.64; with six tiles the work saved weighs as much, 384 columns
// 2.61 and 2.71 ms at 96^3 rows, 0.98 and 0.92 at 64^3, and with five more, 300 columns at 64^3
// 0.69 and 0.65).
constexpr int kGramTilesWhole = 7;
constexpr long kGramTarget = 1024;
static int gram_f64_waves(int npairs) { return npairs <= kGramPairsW4 ? kGramWaves : 1; }
static int gram_f64_nsplit(int npairs, long ng, int most) {
    if (gram_f64_waves(npairs) == 1) return most;
    const long ns = std::min(kGramTarget / npairs, (ng + 255) / 256);
    return (int)std::max(1L, std::min(ns, (long)most));
}

size_t gram_part_elems(int n, int nsplit) { return (size_t)nsplit * 4 * n * n; }

static hipError_t gram_reduce(double *part, int nn, int nsplit, double w, double *G,
                              hipStream_t st) {
    const long blocks = ((long)nn * nn + 63) / 64;
    hipLaunchKernelGGL(k_gram_reduce, dim3((unsigned)blocks), dim3(64 * kRedWaves), 0, st, part, nn,
                       nsplit, w, G);
    return hipGetLastError();
}

hipError_t launch_gram_f64(const double *X, const double *Y, long ld, long ng, int n, double w,
                           double *part, int nsplit, double *G, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int nt = (2 * n + TM - 1) / TM;
    const int npairs = nt * (nt + 1) / 2;
    nsplit = gram_f64_nsplit(npairs, ng, nsplit);
    long kchunk = (ng + nsplit - 1) / nsplit;
    kchunk = (kchunk + 31) / 32 * 32;
    const int vec_ok = (ld % 2 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0) &&
                       ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
    if (nt >= kGramTilesWhole)
        hipLaunchKernelGGL((k_gram_f64<1, true>), dim3(npairs, nsplit), dim3(64), 0, st, X, Y, ld, ng, n,
                           kchunk, part, vec_ok);
    else if (gram_f64_waves(npairs) == 1)
        hipLaunchKernelGGL(k_gram_f64<1>, dim3(npairs, nsplit), dim3(64), 0, st, X, Y, ld, ng, n,
                           kchunk, part, vec_ok);
    else
        hipLaunchKernelGGL(k_gram_f64<kGramWaves>, dim3(npairs, nsplit), dim3(64 * kGramWaves),
                           kGramLds, st, X, Y, ld, ng, n, kchunk, part, vec_ok);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return gram_reduce(part, 2 * n, nsplit, w, G, st);
}

hipError_t launch_gram_cross_f64(const double *X, const double *Y, long ld, long ng, int n,
                                 double w, double *part, int nsplit, double *G, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int nt = (n + TM - 1) / TM;
    nsplit = gram_f64_nsplit(nt * nt, ng, nsplit);
    long kchunk = (ng + nsplit - 1) / nsplit;
    kchunk = (kchunk + 31) / 32 * 32;
    const int vec_ok = (ld % 2 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0) &&
                       ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
    if (gram_f64_waves(nt * nt) == 1)
        hipLaunchKernelGGL(k_gram_cross_f64<1>, dim3(nt * nt, nsplit), dim3(64), 0, st, X, Y, ld, ng,
                           n, kchunk, part, vec_ok);
    else
        hipLaunchKernelGGL(k_gram_cross_f64<kGramWaves>, dim3(nt * nt, nsplit),
                           dim3(64 * kGramWaves), kGramLds, st, X, Y, ld, ng, n, kchunk, part,
                           vec_ok);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long blocks = ((long)n * n + 63) / 64;
    hipLaunchKernelGGL(k_gram_cross_reduce, dim3((unsigned)blocks), dim3(64 * kRedWaves), 0, st,
                       part, n, nsplit, w, G);
    return hipGetLastError();
}

hipError_t launch_gram_bf16(const double *X, const double *Y, long ld, long ng, int n, double w,
                            double *part, int nsplit, double *G, __bf16 *zx, __bf16 *zy,
                            bool pack_x, bool pack_y, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    // BF16 rows are read in whole 32-row steps of 16-byte loads: ld a multiple of 32,
    // 16-byte aligned operands
    if (ld % 32 != 0 || (reinterpret_cast<uintptr_t>(X) & 15) || (reinterpret_cast<uintptr_t>(Y) & 15) ||
        (reinterpret_cast<uintptr_t>(zx) & 15) || (reinterpret_cast<uintptr_t>(zy) & 15))
        return hipErrorInvalidValue;
    const long items = (long)n * (ld / 8);
    long blocks = (items + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipError_t e;
    if (pack_x) {
        hipLaunchKernelGGL(k_pack_bf16, dim3((unsigned)blocks), dim3(256), 0, st, X, ld, ng, n, zx);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (pack_y) {
        hipLaunchKernelGGL(k_pack_bf16, dim3((unsigned)blocks), dim3(256), 0, st, Y, ld, ng, n, zy);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // one 1024-thread workgroup per CU: enough K-chunks for one round over 256 CUs
    const int nst = (2 * n + kSuper - 1) / kSuper;
    const int nsp = nst * (nst + 1) / 2;
    nsplit = max(1, min(nsplit, 256 / nsp));
    long kchunk = (ng + nsplit - 1) / nsplit;
    kchunk = (kchunk + 31) / 32 * 32;
    hipLaunchKernelGGL(k_gram_bf16_super, dim3(nsp, nsplit), dim3(1024), 0, st, zx, zy, ld, ng, n,
                       kchunk, part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return gram_reduce(part, 2 * n, nsplit, w, G, st);
}

}  // namespace qo
