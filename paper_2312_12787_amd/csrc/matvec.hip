// matvec.hip -- dense complex products Y = A X of the GMRES solve (Sec. 3.2:
// every Krylov step costs one product with the dense collocation matrix) and
// the residual R = B - A X with FP64 accumulation.
//
// Layouts: A column-major (lda); X, Y column-major blocks, one column per
// right-hand side.  Up to 4 right-hand sides: VALU kernel (k_matvec); more:
// matrix-core kernel (k_matvec_mfma), up to 64 right-hand sides per pass over A.  Both split the columns over blocks and
// add the split partial sums in a fixed order (k_matvec_reduce).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "../../include/bem.h"
#include "internal.h"
#include "krylov_dev.h"
#include "launch.h"

namespace bemk {

int matvec_splits_valu(int n);

namespace {

constexpr int BS = 256;        // threads per block
constexpr int MV_WAVES = 4;    // row tiles per block (64 rows each for VALU, 16 for MFMA)
constexpr int MV_CH = 32;      // X columns staged in LDS per step (VALU kernel)

// ---------------------------------------------------------------------------
// Dense complex product Y = A X, split over columns.  A block holds four waves;
// each wave owns 64 consecutive rows (one row per lane: coalesced 1 KiB loads of
// a column-major A) and the block shares the X values of its column range
// through LDS.  Partial sums of each column split go to `part` and are added
// in split order by k_matvec_reduce.  TA / TX: storage types (double2 or
// float2); ACC: accumulation type.
// ---------------------------------------------------------------------------
// The matrix is streamed once per product and is larger than the caches:
// non-temporal loads keep it from displacing the reused X blocks (measured on
// gfx950: 2.7 % faster FP64 products at n = 8192, 16 right-hand sides).
template <class TA>
__device__ __forceinline__ TA ld_stream(const TA* p)
{
    TA v;
    v.x = __builtin_nontemporal_load(&p->x);
    v.y = __builtin_nontemporal_load(&p->y);
    return v;
}

template <int NR, class TA, class TX, class ACC>
__global__ __launch_bounds__(BS) void k_matvec(const TA* __restrict__ A, size_t lda, int n,
                                               const TX* __restrict__ X, size_t ldx, int nrhs,
                                               ACC* __restrict__ part, int cps)
{
    using S = decltype(ACC{}.x);
    __shared__ ACC xs[MV_CH][NR];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = (blockIdx.x * MV_WAVES + wave) * 64 + lane;
    const int c0 = blockIdx.y * cps;
    const int c1 = min(n, c0 + cps);
    S ar[NR], ai[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) ar[r] = ai[r] = S(0);
    for (int cb = c0; cb < c1; cb += MV_CH) {
        const int nc = min(MV_CH, c1 - cb);
        __syncthreads();
        for (int t = threadIdx.x; t < MV_CH * NR; t += BS) {
            const int c = t % MV_CH, r = t / MV_CH;
            ACC v;
            v.x = S(0);
            v.y = S(0);
            if (c < nc && r < nrhs) {
                const TX x = X[(size_t)r * ldx + cb + c];
                v.x = (S)x.x;
                v.y = (S)x.y;
            }
            xs[c][r] = v;
        }
        __syncthreads();
        if (row < n) {
            const TA* ap = A + (size_t)cb * lda + row;
            if (nc == MV_CH) {
#pragma unroll 8
                for (int c = 0; c < MV_CH; ++c) {
                    const TA a = ld_stream(ap + (size_t)c * lda);
                    const S axr = (S)a.x, axi = (S)a.y;
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        const ACC x = xs[c][r];
                        ar[r] = fma(axr, x.x, ar[r]);
                        ar[r] = fma(-axi, x.y, ar[r]);
                        ai[r] = fma(axr, x.y, ai[r]);
                        ai[r] = fma(axi, x.x, ai[r]);
                    }
                }
            } else {
                for (int c = 0; c < nc; ++c) {
                    const TA a = ld_stream(ap + (size_t)c * lda);
                    const S axr = (S)a.x, axi = (S)a.y;
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        const ACC x = xs[c][r];
                        ar[r] = fma(axr, x.x, ar[r]);
                        ar[r] = fma(-axi, x.y, ar[r]);
                        ai[r] = fma(axr, x.y, ai[r]);
                        ai[r] = fma(axi, x.x, ai[r]);
                    }
                }
            }
        }
    }
    if (row < n) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
            if (r < nrhs) {
                ACC v;
                v.x = ar[r];
                v.y = ai[r];
                part[((size_t)blockIdx.y * nrhs + r) * n + row] = v;
            }
    }
}

// Y[:, r] = sum over splits (in order, in FP64) of the partial products; optionally
// R = B - Y (residual form) when B != nullptr.
template <class ACC, class TY>
__global__ void k_matvec_reduce(const ACC* __restrict__ part, int splits, int n, int nrhs, TY* __restrict__ Y,
                                size_t ldy, const double2* __restrict__ B, size_t ldb)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (row >= n || r >= nrhs) return;
    double sr = 0.0, si = 0.0;
    for (int s = 0; s < splits; ++s) {
        const ACC v = part[((size_t)s * nrhs + r) * n + row];
        sr += v.x;
        si += v.y;
    }
    TY out;
    if (B) {
        const double2 b = B[(size_t)r * ldb + row];
        out.x = (decltype(out.x))(b.x - sr);
        out.y = (decltype(out.y))(b.y - si);
    } else {
        out.x = (decltype(out.x))sr;
        out.y = (decltype(out.y))si;
    }
    Y[(size_t)r * ldy + row] = out;
}


// ---------------------------------------------------------------------------
// Block product on the matrix cores (more than 4 right-hand sides).  The
// complex product is four real products, Yr = Ar Xr + Ai (-Xi), Yi = Ar Xi +
// Ai Xr, each a 16 x 16 x 4 MFMA: one wave owns 16 rows and walks its column
// range 4 columns at a time; lane l holds A[row0 + l % 16][c + l / 16] and
// X[c + l / 16][rhs = l % 16] (X packed right-hand-side fastest, XT[c * 16 + r]),
// and receives result j = 0..3 at row row0 + 4 (l / 16) + j (FP32 MFMA) or
// row0 + (l / 16) + 4 j (FP64 MFMA), right-hand side l % 16 (lane layouts
// checked on gfx950).  No LDS, no broadcast: every lane loads its own operands.
// ---------------------------------------------------------------------------
typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <class T>
struct Mfma;
template <>
struct Mfma<double> {
    using acc = d4v;
    using v2 = double2;
    static __device__ __forceinline__ int out_row(int lk, int j) { return lk + 4 * j; }
    static __device__ __forceinline__ acc run(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};
template <>
struct Mfma<float> {
    using acc = f4v;
    using v2 = float2;
    static __device__ __forceinline__ int out_row(int lk, int j) { return 4 * lk + j; }
    static __device__ __forceinline__ acc run(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

// RT: 16-row tiles per wave (they share each X load); U: column steps in flight;
// G3: complex product with three real products (P1 = Ar Xr, P2 = Ai Xi,
// P3 = (Ar + Ai)(Xr + Xi); Yr = P1 - P2, Yi = P3 - P1 - P2) instead of four;
// NG: groups of 16 right-hand sides taken in the same pass over A (X packed
// XT[c * 16 NG + r]), so that one read of A serves up to 64 right-hand sides.
// The wide shapes, which are matrix-core bound, carry an occupancy target:
// left alone the compiler puts their accumulators in AGPRs beside the load
// slots and runs one or two waves per SIMD; with the target they fit in the
// VGPRs (FP32 sums over three or four groups, with their totals: two waves;
// FP64 sums over two to four groups, where RT * NG <= 4 keeps them spill-free:
// two waves, the kite16384 FP64 path 73.7 -> 84.4 solves/s).  The single-group shapes keep the compiler's
// own allocation (the HBM-bound 16-RHS product pipelines its loads instead).
constexpr int mfma_min_waves(int tbytes, int rt, int ng)
{
    return (tbytes == 4 && ng >= 3) ? 2 : (tbytes == 8 && ng >= 2 && rt * ng <= 4) ? 2 : 1;
}

template <class TA, class T, int RT, int U, bool G3, int NG>
__global__ __launch_bounds__(BS, mfma_min_waves(sizeof(T), RT, NG)) void k_matvec_mfma(const TA* __restrict__ A, size_t lda, int n,
                                                    const typename Mfma<T>::v2* __restrict__ XT, int nrhs,
                                                    typename Mfma<T>::v2* __restrict__ part, int cps)
{
    using M = Mfma<T>;
    using acc = typename M::acc;
    using V2 = typename M::v2;
    constexpr int XW = 16 * NG;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lk = lane >> 4;
    const int row0 = (blockIdx.x * MV_WAVES + wave) * 16 * RT;
    bool rok[RT];
    const TA* ap[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int row = row0 + 16 * t + lr;
        rok[t] = row < n;
        ap[t] = A + (rok[t] ? row : 0);
    }
    const int first = blockIdx.y * cps, end = min(n, first + cps);
    acc rr0[NG][RT], rr1[NG][RT], ii0[NG][RT], ii1[NG][RT];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int t = 0; t < RT; ++t) rr0[g][t] = rr1[g][t] = ii0[g][t] = ii1[g][t] = acc{0, 0, 0, 0};
    // The FP32 sums of two and more groups run over 256 columns at most and are
    // then added to totals, so that their rounding does not grow with the
    // columns of a split (n = 16384, 64 right-hand sides, largest error against
    // FP64 sums 1.1e-6 with 8 splits, 2.2e-6 with the faster 2, 4.4e-7 folded).
    // The other shapes have no registers to spare for totals.  The FP64 sums of
    // one group, whose splits group_splits chooses by how they fill the chip, run
    // over an eighth of the columns and are then added to totals in LDS (rms
    // error, kite, 16 random right-hand sides, so / over whole splits: n = 8192
    // 3.2e-14 / 4.6e-14, 16384 8.5e-14 / 1.7e-13).  The pipeline starts anew for
    // each part: n = 8192 171 -> 174 us (totals in registers 188, as more partial
    // sums in memory 189, both what eight splits take).
    constexpr int FOLD = sizeof(T) == 4 && NG >= 2 ? 256 : 0;
    acc sum[4][FOLD ? NG : 1][FOLD ? RT : 1];
    if (FOLD)
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int t = 0; t < RT; ++t) sum[0][g][t] = sum[1][g][t] = sum[2][g][t] = sum[3][g][t] = acc{0, 0, 0, 0};
    auto fold = [&]() {
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                sum[0][g][t] += rr0[g][t];
                sum[1][g][t] += rr1[g][t];
                sum[2][g][t] += ii0[g][t];
                if (!G3) sum[3][g][t] += ii1[g][t];
                rr0[g][t] = rr1[g][t] = ii0[g][t] = ii1[g][t] = acc{0, 0, 0, 0};
            }
    };
    constexpr bool PARTS = sizeof(T) == 8 && NG == 1;
    __shared__ V2 total[PARTS ? RT : 1][PARTS ? 4 : 1][PARTS ? BS : 1];  // a lane reads and writes its own
    // the sum of result j of a row tile
    auto value = [&](int g, int t, int j) {
        V2 v;
        if (G3) {
            v.x = rr0[g][t][j] - rr1[g][t][j];
            v.y = ii0[g][t][j] - rr0[g][t][j] - rr1[g][t][j];
        } else {
            v.x = rr0[g][t][j] + rr1[g][t][j];
            v.y = ii0[g][t][j] + ii1[g][t][j];
        }
        return v;
    };
    // one 16 x 4 tile of A (per row tile) against 4 x 16 NG of X
    auto step = [&](const T (&ar)[RT], const T (&ai)[RT], const T (&xr)[NG], const T (&xi)[NG]) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                if (G3) {
                    rr0[g][t] = M::run(ar[t], xr[g], rr0[g][t]);
                    rr1[g][t] = M::run(ai[t], xi[g], rr1[g][t]);
                    ii0[g][t] = M::run(ar[t] + ai[t], xr[g] + xi[g], ii0[g][t]);
                } else {
                    rr0[g][t] = M::run(ar[t], xr[g], rr0[g][t]);
                    rr1[g][t] = M::run(ai[t], -xi[g], rr1[g][t]);
                    ii0[g][t] = M::run(ar[t], xi[g], ii0[g][t]);
                    ii1[g][t] = M::run(ai[t], xr[g], ii1[g][t]);
                }
            }
    };
    // HBM-bound shapes (one group of 16 right-hand sides, at most 16 tile
    // loads per step) walk the columns software-pipelined: the loads of the
    // next 4U columns are issued before the products of the current ones, so
    // a wave keeps its reads in flight while its matrix-core work runs.  The
    // wider shapes, matrix-core bound, would spill a second buffer; they
    // rotate their slots instead (below).
    constexpr bool PIPE = NG == 1 && RT * U <= 16;
    auto load = [&](TA (&a)[U][RT], V2 (&x)[U][NG], int cc) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = cc + 4 * u + lk;
#pragma unroll
            for (int g = 0; g < NG; ++g) x[u][g] = XT[(size_t)col * XW + 16 * g + lr];
#pragma unroll
            for (int t = 0; t < RT; ++t) a[u][t] = ld_stream(ap[t] + (size_t)col * lda);
        }
    };
    auto compute = [&](const TA (&a)[U][RT], const V2 (&x)[U][NG]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            T ar[RT], ai[RT], xr[NG], xi[NG];
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                ar[t] = rok[t] ? (T)a[u][t].x : T(0);
                ai[t] = rok[t] ? (T)a[u][t].y : T(0);
            }
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                xr[g] = x[u][g].x;
                xi[g] = x[u][g].y;
            }
            step(ar, ai, xr, xi);
        }
    };
    // (a multiple of every 4U)
    const int cols = PARTS ? ((n + 7) / 8 + 31) / 32 * 32 : cps;
    int c0 = first;
    do {  // once at least: a split without columns leaves zeros
        const int c1 = min(end, c0 + cols);
        int c = c0;
        if constexpr (!PIPE) {
            // rotating slots: slot u of the next 4U columns is loaded as soon as
            // slot u of the current ones has gone into the matrix cores, so a
            // wave keeps loads in flight without a second buffer; the scheduling
            // barriers keep that order (the compiler otherwise moves the loads
            // next to their uses and waits for all of them).  Measured on gfx950,
            // kite of 16384 elements, 64 right-hand sides: FP32 product 3.82 ->
            // 3.50 ms at the same register count (two waves per SIMD)
            if (c + 4 * U <= c1) {
                TA a[U][RT];
                V2 x[U][NG];
                load(a, x, c);
                for (;;) {
                    const int cn = c + 4 * U;
                    const bool more = cn + 4 * U <= c1;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        T ar[RT], ai[RT], xr[NG], xi[NG];
#pragma unroll
                        for (int t = 0; t < RT; ++t) {
                            ar[t] = rok[t] ? (T)a[u][t].x : T(0);
                            ai[t] = rok[t] ? (T)a[u][t].y : T(0);
                        }
#pragma unroll
                        for (int g = 0; g < NG; ++g) {
                            xr[g] = x[u][g].x;
                            xi[g] = x[u][g].y;
                        }
                        step(ar, ai, xr, xi);
                        __builtin_amdgcn_sched_barrier(0);
                        // unconditional (the last pass reloads its own columns):
                        // a load under a branch makes the compiler wait for every
                        // load in flight before the next slot
                        const int col = (more ? cn : c) + 4 * u + lk;
#pragma unroll
                        for (int g = 0; g < NG; ++g) x[u][g] = XT[(size_t)col * XW + 16 * g + lr];
#pragma unroll
                        for (int t = 0; t < RT; ++t) a[u][t] = ld_stream(ap[t] + (size_t)col * lda);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    c = cn;
                    if constexpr (FOLD != 0)
                        if ((c - c0) % FOLD == 0) fold();
                    if (!more) break;
                }
            }
        } else if (c + 4 * U <= c1) {
            TA a[U][RT];
            V2 x[U][NG];
            load(a, x, c);
            for (;;) {
                const int cn = c + 4 * U;
                if (cn + 4 * U > c1) {
                    compute(a, x);
                    c = cn;
                    break;
                }
                TA an[U][RT];
                V2 xn[U][NG];
                load(an, xn, cn);
                compute(a, x);
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int t = 0; t < RT; ++t) a[u][t] = an[u][t];
#pragma unroll
                    for (int g = 0; g < NG; ++g) x[u][g] = xn[u][g];
                }
                c = cn;
            }
        }
        for (; c < c1; c += 4) {
            const int col = c + lk;
            const bool ok = col < c1;
            T ar[RT], ai[RT], xr[NG], xi[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                xr[g] = T(0);
                xi[g] = T(0);
                if (ok) {
                    const V2 x = XT[(size_t)col * XW + 16 * g + lr];
                    xr[g] = x.x;
                    xi[g] = x.y;
                }
            }
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                ar[t] = T(0);
                ai[t] = T(0);
                if (ok && rok[t]) {
                    const TA a = ld_stream(ap[t] + (size_t)col * lda);
                    ar[t] = (T)a.x;
                    ai[t] = (T)a.y;
                }
            }
            step(ar, ai, xr, xi);
        }
        if constexpr (FOLD != 0) {
            fold();
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    rr0[g][t] = sum[0][g][t];
                    rr1[g][t] = sum[1][g][t];
                    ii0[g][t] = sum[2][g][t];
                    ii1[g][t] = sum[3][g][t];
                }
        }
        if (PARTS && end - first > cols) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    V2 v = value(0, t, j);
                    if (c0 != first) {
                        const V2 before = total[t][j][threadIdx.x];
                        v.x += before.x;
                        v.y += before.y;
                    }
                    total[t][j][threadIdx.x] = v;
                }
                rr0[0][t] = rr1[0][t] = ii0[0][t] = ii1[0][t] = acc{0, 0, 0, 0};
            }
        }
        c0 += cols;
    } while (PARTS && c0 < end);
    const bool totals = PARTS && end - first > cols;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int r = 16 * g + lr;
        if (r >= nrhs) continue;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = row0 + 16 * t + M::out_row(lk, j);
                if (row < n)
                    part[((size_t)blockIdx.y * nrhs + r) * n + row] = totals ? total[t][j][threadIdx.x] : value(g, t, j);
            }
    }
}

// ---------------------------------------------------------------------------
// Row-block products: one workgroup owns 16 rows and ALL columns, its waves
// take the column groups in turn and add their sums through LDS in wave order,
// so a product is one launch: no split partial sums in memory, no reduction
// pass, and (bem_matvec) X read where it lies instead of packed first.  For
// systems small enough that launches and idle compute units, not HBM, set the
// time: a product split over columns needs two to three launches, and its
// built-in shapes fill 64 to 128 of 256 CUs at n = 1024 .. 2048.  The matrix
// stays in the Infinity Cache, so its loads are ordinary ones (non-temporal
// ones made the 16-right-hand-side product of n = 1554 25.3 instead of 20.8
// us).  Bound by one CU's read and FP64 matrix rate (a block of 16 rows has
// 1/97 of the work at n = 1554) and by the chain load - product - LDS sum -
// store.
// ---------------------------------------------------------------------------
enum RowMode { ROW_PRODUCT, ROW_RESIDUAL, ROW_STEP };

// What becomes of the sums: Y = A X, R = B - A X, or the Krylov step's product
// with the previous vector's normalisation (see k_step_reduce).
template <class TY, class TV>
struct RowOut {
    TY* Y;
    size_t ldy;
    const double2* B;
    size_t ldb;
    const double* nrm;
    int nu;
    TV* V;
    size_t ldv;
    double* hnorm;
    int* active;
};

constexpr int ROW_MAX_WAVES = 16;

// Row tile of this block.  Blocks go to the eight XCDs in turn.  Where columns
// do not start on 128-byte lines, neighbouring tiles go to the same XCD, so that
// the line they share is brought into one L2 (mixed request, n = 2674 with lda =
// n: 12.65 -> 11.98 ms); aligned columns share none and stay in block order
// (n = 1554, lda 1560: 14.2 us, grouped 14.4).
__device__ __forceinline__ int row_tile(size_t lda, size_t entry)
{
    if ((lda * entry & 127) == 0) return blockIdx.x;
    return ((int)blockIdx.x & 7) * ((int)gridDim.x / 8) + ((int)blockIdx.x >> 3);
}

// |w| of the step's right-hand sides: wave w takes r = w, w + nw; the loads go
// out before the product, the sums are formed after it.
struct StepScale {
    double part[2];
    template <class O>
    __device__ __forceinline__ void load(const O& o, int wave, int nw, int nr)
    {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            part[k] = 0.0;
            const int r = wave + k * nw;
            if (r < nr)
                for (int b = threadIdx.x & 63; b < o.nu; b += 64) part[k] += o.nrm[(size_t)r * o.nu + b];
        }
    }
    template <class O>
    __device__ __forceinline__ void finish(const O& o, int wave, int nw, int nr, double* inv_s, int* act_s) const
    {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int r = wave + k * nw;
            if (r >= nr) continue;
            const double beta = sqrt(dev::wave_sum(part[k]));
            if ((threadIdx.x & 63) == 0) {
                const int act = o.active[r];
                inv_s[r] = dev::inv_beta(beta);
                act_s[r] = act;
                if (blockIdx.x == 0) {
                    if (act == 1) o.hnorm[r] = beta;
                    // every block of a marked column skips it, whether it reads the mark or the zero
                    if (act == dev::STOPPING) o.active[r] = 0;
                }
            }
        }
    }
};

__device__ __forceinline__ void st_row(double2* p, double2 v) { *p = v; }
__device__ __forceinline__ void st_row(float2* p, double2 v) { *p = make_float2((float)v.x, (float)v.y); }

template <int MODE, class O>
__device__ __forceinline__ void row_store(const O& o, int row, int r, double sr, double si, const double* inv_s,
                                          const int* act_s)
{
    auto* y = o.Y + (size_t)r * o.ldy + row;
    if (MODE == ROW_RESIDUAL) {
        const double2 b = o.B[(size_t)r * o.ldb + row];
        sr = b.x - sr;
        si = b.y - si;
    } else if (MODE == ROW_STEP) {
        const double inv = inv_s[r];
        const double2 w = make_double2(y->x, y->y);
        if (act_s[r] == 1) st_row(o.V + (size_t)r * o.ldv + row, make_double2(w.x * inv, w.y * inv));
        sr *= inv;
        si *= inv;
    }
    st_row(y, make_double2(sr, si));
}

// Matrix-core form, 5 to 16 right-hand sides: operand layout, 3-product form
// and result rows as k_matvec_mfma's; the loads of a wave's next 4U columns go
// out before the products of the current ones.  PACKED: X is XT[c * 16 + r],
// else column-major (ldx).
template <class TA, class T, class TX, int U, bool PACKED, int MODE, class O>
__global__ __launch_bounds__(64 * ROW_MAX_WAVES) void k_rowblock_mfma(const TA* __restrict__ A, size_t lda, int n,
                                                                      const TX* __restrict__ X, size_t ldx, int nrhs,
                                                                      const O o)
{
    using M = Mfma<T>;
    using acc = typename M::acc;
    extern __shared__ double row_lds[];
    __shared__ double inv_s[16];
    __shared__ int act_s[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int row0 = row_tile(lda, sizeof(TA)) * 16;
    if (row0 >= n) return;
    const TA* ap = A + min(row0 + lr, n - 1);
    const TX* xp = PACKED ? X + lr : X + (size_t)min(lr, nrhs - 1) * ldx;
    StepScale sc;
    if (MODE == ROW_STEP) sc.load(o, wave, nw, nrhs);
    acc rr0{0, 0, 0, 0}, rr1{0, 0, 0, 0}, ii{0, 0, 0, 0};
    auto load = [&](TA (&a)[U], TX (&x)[U], int c) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = min(c + 4 * u + lk, n - 1);
            x[u] = PACKED ? xp[(size_t)col * 16] : xp[col];
            a[u] = ap[(size_t)col * lda];
        }
    };
    auto compute = [&](const TA (&a)[U], const TX (&x)[U], int c) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = c + 4 * u + lk < n;
            const T ar = ok ? (T)a[u].x : T(0), ai = ok ? (T)a[u].y : T(0);
            const T xr = ok ? (T)x[u].x : T(0), xi = ok ? (T)x[u].y : T(0);
            rr0 = M::run(ar, xr, rr0);
            rr1 = M::run(ai, xi, rr1);
            ii = M::run(ar + ai, xr + xi, ii);
        }
    };
    // FP32 sums over 256 columns at most, then into totals, as k_matvec_mfma's
    constexpr int FOLD = sizeof(T) == 4 ? 256 / (4 * U) : 0;
    acc s0{0, 0, 0, 0}, s1{0, 0, 0, 0}, s2{0, 0, 0, 0};
    int c = wave * 4 * U;
    if (c < n) {
        TA a[U];
        TX x[U];
        load(a, x, c);
        for (int trip = 1;; ++trip) {
            const int cn = c + nw * 4 * U;
            if (cn >= n) {
                compute(a, x, c);
                break;
            }
            TA an[U];
            TX xn[U];
            load(an, xn, cn);
            compute(a, x, c);
            if constexpr (FOLD != 0)
                if (trip % FOLD == 0) {
                    s0 += rr0;
                    s1 += rr1;
                    s2 += ii;
                    rr0 = rr1 = ii = acc{0, 0, 0, 0};
                }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = an[u];
                x[u] = xn[u];
            }
            c = cn;
        }
    }
    if (FOLD != 0) {
        rr0 += s0;
        rr1 += s1;
        ii += s2;
    }
    T* red = reinterpret_cast<T*>(row_lds);  // [wave][2 j + part][lane]
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        red[(wave * 8 + 2 * j) * 64 + lane] = rr0[j] - rr1[j];
        red[(wave * 8 + 2 * j + 1) * 64 + lane] = ii[j] - rr0[j] - rr1[j];
    }
    if (MODE == ROW_STEP) sc.finish(o, wave, nw, nrhs, inv_s, act_s);
    __syncthreads();
    const int t = threadIdx.x, rl = t & 15, r = t >> 4;  // thread: row rl, right-hand side r
    const int row = row0 + rl;
    if (t >= 256 || r >= nrhs || row >= n) return;
    // the lane and element that hold row rl of right-hand side r
    const bool f64 = sizeof(T) == 8;
    const int j = f64 ? rl >> 2 : rl & 3, src = (f64 ? rl & 3 : rl >> 2) * 16 + r;
    double sr = 0.0, si = 0.0;
    for (int w = 0; w < nw; ++w) {
        sr += red[(w * 8 + 2 * j) * 64 + src];
        si += red[(w * 8 + 2 * j + 1) * 64 + src];
    }
    row_store<MODE>(o, row, r, sr, si, inv_s, act_s);
}

// Vector form, NR = 1 to 4 right-hand sides: lane l holds row l % 16 and column
// l / 16 of each 16 x 4 tile.  All of X goes to LDS first (from global memory a
// wave's read of one value of X costs as much of the L1's rate as its read of a
// tile of A).  PACKED: X is XT[c * NR + r].
template <int NR, class TA, class TX, class ACC, int U, bool PACKED, int MODE, class O>
__global__ __launch_bounds__(64 * ROW_MAX_WAVES) void k_rowblock_vec(const TA* __restrict__ A, size_t lda, int n,
                                                                     const TX* __restrict__ X, size_t ldx, const O o)
{
    using S = decltype(ACC{}.x);
    extern __shared__ double row_lds[];
    ACC* xs = reinterpret_cast<ACC*>(row_lds);  // [column][NR]
    __shared__ S red[ROW_MAX_WAVES][2 * NR][16];
    __shared__ double inv_s[4];
    __shared__ int act_s[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int row0 = row_tile(lda, sizeof(TA)) * 16;
    if (row0 >= n) return;
    const TA* ap = A + min(row0 + lr, n - 1);
    StepScale sc;
    if (MODE == ROW_STEP) sc.load(o, wave, nw, NR);
    auto load = [&](TA (&a)[U], int c) {
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = ap[(size_t)min(c + 4 * u + lk, n - 1) * lda];
    };
    int c = wave * 4 * U;
    TA a[U];
    if (c < n) load(a, c);
    for (int t = threadIdx.x; t < n * NR; t += blockDim.x) {
        const int r = PACKED ? 0 : t / n;
        const TX x = PACKED ? X[t] : X[(size_t)r * ldx + (t - r * n)];
        ACC v;
        v.x = (S)x.x;
        v.y = (S)x.y;
        xs[PACKED ? t : (t - r * n) * NR + r] = v;
    }
    __syncthreads();
    S ar[NR], ai[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) ar[r] = ai[r] = S(0);
    while (c < n) {
        const int cn = c + nw * 4 * U;
        TA an[U];
        if (cn < n) load(an, cn);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int col = c + 4 * u + lk;
            const bool ok = col < n;
            const S axr = ok ? (S)a[u].x : S(0), axi = ok ? (S)a[u].y : S(0);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const ACC x = xs[min(col, n - 1) * NR + r];
                const S xr = ok ? x.x : S(0), xi = ok ? x.y : S(0);
                ar[r] = fma(axr, xr, ar[r]);
                ar[r] = fma(-axi, xi, ar[r]);
                ai[r] = fma(axr, xi, ai[r]);
                ai[r] = fma(axi, xr, ai[r]);
            }
        }
        if (cn >= n) break;
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = an[u];
        c = cn;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        ar[r] += __shfl_xor(ar[r], 16, 64);
        ai[r] += __shfl_xor(ai[r], 16, 64);
        ar[r] += __shfl_xor(ar[r], 32, 64);
        ai[r] += __shfl_xor(ai[r], 32, 64);
        if (lk == 0) {
            red[wave][2 * r][lr] = ar[r];
            red[wave][2 * r + 1][lr] = ai[r];
        }
    }
    if (MODE == ROW_STEP) sc.finish(o, wave, nw, NR, inv_s, act_s);
    __syncthreads();
    const int t = threadIdx.x, rl = t & 15, r = t >> 4;
    const int row = row0 + rl;
    if (r >= NR || row >= n) return;
    double sr = 0.0, si = 0.0;
    for (int w = 0; w < nw; ++w) {
        sr += red[w][2 * r][rl];
        si += red[w][2 * r + 1][rl];
    }
    row_store<MODE>(o, row, r, sr, si, inv_s, act_s);
}

// X of a row-block vector product fits the LDS beside the wave sums.
constexpr size_t ROW_X_BYTES = 128 * 1024;
bool row_fits(int n, int nr, size_t value_bytes) { return nr > 4 || (size_t)n * nr * value_bytes <= ROW_X_BYTES; }

// A row-block product of up to 16 right-hand sides.  16 waves per workgroup
// where the rows alone leave the chip's CUs less than one workgroup each, and in
// the vector form always: a lane sums 1/64 of the columns then, as much as the
// 64 splits of the split form (FP32, 3 right-hand sides, n = 4800, 8 / 16 waves:
// rms error 4.2e-6 / 3.0e-6, 59 / 51 us).
template <class TA, class TX, class ACC, bool PACKED, int MODE, class O>
void launch_rowblock(const TA* A, size_t lda, int n, const TX* X, size_t ldx, int nr, const O& o, hipStream_t s)
{
    using S = decltype(ACC{}.x);
    const int tiles = (n + 15) / 16, nw = tiles <= 256 || nr <= 4 ? 16 : 8;
    const int blocks = (tiles + 7) / 8 * 8;  // see row_tile
    constexpr int U = sizeof(TA) == 16 || sizeof(S) == 8 ? 4 : 8;
    const size_t xlds = (size_t)n * nr * sizeof(ACC);
#define BEM_ROW_VEC(NR_)                                                                                              \
    hipLaunchKernelGGL((k_rowblock_vec<NR_, TA, TX, ACC, U, PACKED, MODE, O>), dim3(blocks), dim3(64 * nw), xlds, s, A, \
                       lda, n, X, ldx, o)
    if (nr > 4)
        hipLaunchKernelGGL((k_rowblock_mfma<TA, S, TX, U, PACKED, MODE, O>), dim3(blocks), dim3(64 * nw),
                           (size_t)nw * 8 * 64 * sizeof(S), s, A, lda, n, X, ldx, nr, o);
    else if (nr == 1)
        BEM_ROW_VEC(1);
    else if (nr == 2)
        BEM_ROW_VEC(2);
    else if (nr == 3)
        BEM_ROW_VEC(3);
    else
        BEM_ROW_VEC(4);
#undef BEM_ROW_VEC
}

// XT[c * xw + r] = X[r * ldx + c] (r < nr), 0 for nr <= r < xw (xw = 16, 32, 48, 64)
template <class TX, class V2>
__global__ void k_pack_xt(const TX* __restrict__ X, size_t ldx, int n, int nr, int xw, V2* __restrict__ XT)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = t / xw, r = t - c * xw;
    if (c >= n) return;
    V2 v;
    v.x = 0;
    v.y = 0;
    if (r < nr) {
        const TX x = X[(size_t)r * ldx + c];
        v.x = x.x;
        v.y = x.y;
    }
    XT[(size_t)c * xw + r] = v;
}

// Column splits of the FP64 product over one group of 16 right-hand sides, with
// rows split into blocks of 128.  256 blocks run at once, one per CU (the
// registers leave one wave per SIMD).  More go in another turn, which costs as
// much as a full one, and each split writes and re-reads its partial sums: the
// fewest splits that fill the turns they take to 4/5.
int group_splits(int n)
{
    const int rowblocks = (n + 127) / 128, most = std::max(1, std::min(64, n / 64));
    int best = 1;
    double fill = 0;
    for (int s = 1; s <= most && fill < 0.8; ++s) {
        const int blocks = rowblocks * s, turns = (blocks + 255) / 256;
        const double f = (double)blocks / (256.0 * turns);
        if (f > fill) {
            fill = f;
            best = s;
        }
    }
    return best;
}

// Column splits of the product over 2-4 groups, which is bound by the matrix
// cores: a CU's blocks share them, so the fullest CU sets the time, ceil(blocks
// / 256) blocks of n / splits columns; a block costs about 40 columns more to
// start and to end.  A lone wave per SIMD with FP64 sums over one row tile
// leaves gaps (5 %; two row tiles, or FP32 sums, have twice the products in a
// step and none).
//
// FP64 sums, which run through a whole split, take `least_splits` or more.
int wide_splits(int n, int rt, bool f64, int least_splits, int most)
{
    const int rowblocks = (n + 16 * rt * MV_WAVES - 1) / (16 * rt * MV_WAVES);
    const int first = std::min(least_splits, most);
    int best = first;
    double least = 0;
    for (int s = first; s <= most; ++s) {
        const int deep = (rowblocks * s + 255) / 256;
        double cost = deep * (1.0 / s + 40.0 / n);
        if (f64 && rt == 1 && deep == 1) cost *= 1.05;
        if (s == first || cost < least) {
            least = cost;
            best = s;
        }
    }
    return best;
}

// The most column splits a product may take: its partial-sum buffer is sized for them.
int split_limit(int n, int ng)
{
    const int want = (131072 + n - 1) / std::max(1, n);  // about 2048 blocks at one row tile per wave
    return std::max(1, std::min({ng <= 2 ? std::max(want, 8) : want, 64, std::max(1, n / 64)}));
}

// Launch shape of the matrix-core product: row tiles per wave, column steps
// in flight, column splits, 3-product form, for one group of 16 right-hand
// sides and for 2-4 groups per pass.
//
// One group (bem_matvec, 16 right-hand sides, us).  FP64, ten calls back to back, 8
// splits at every size / group_splits: n 4400 91 / 80, 5400 119 / 104, 8192 195 /
// 192 (a call among others 187 / 174), 10000 311 / 274, 12000 394 / 392, 16384
// 702 / 657.  FP32 keeps 8 splits (fewer are
// up to 15 % faster, but long FP32 sums lose accuracy), 8 / 4 column steps in
// flight: n 6800 90.2 / 86.7, 8192 106 / 104, 12000 232 / 218, 16384 412 / 405.
//
// 2-4 groups (32, 48 and 64 right-hand sides, us; splits for about 1024 blocks,
// FP32 and two groups of FP64 always 2 and 1 row tiles / as here): FP32 n 1554
// 28.8, 36.3, 45.2 / 20.0, 23.9, 27.1; 2674  33.5, 42.9, 50.5 / 31.6, 37.5, 44.9;
// 4096  52.1, 64.8, 81.5 / 47.0, 61.6, 74.0; 10000  237, 325, 438 / 220, 294, 374;
// 16384  533, 715, 957 / 511, 686, 886; FP64 n 1554  27.2, 37.1, 44.3 / 24.9, 30.5,
// 34.7; 2674  54.2, 62.6, 77.4 / 44.6, 55.0, 68; 6000  156, 209, 272 / 146, 203,
// 261; 10000  416, 550, 712 / 374, 508, 651; 16384  1026, 1285, 1618 / 919, 1278,
// 1612.  Two row tiles read X half as often, but fill the chip with longer
// splits: below n = 3072 one is faster (FP32, 64 right-hand sides, best
// splits of each, 1 / 2 tiles: n 2674 44.9 / 47.4, 4096 79.4 / 74.0; FP64, 32:
// 42.0 / 42.7, 74.6 / 72.7).  FP64 sums over 3-4 groups take one, whose registers
// leave two waves per SIMD (n = 8192, 64 right-hand sides: 425 / 503).
MvShape mfma_default(int n, int ng, bool f64)
{
    const int most = split_limit(n, ng);
    if (ng == 1) return f64 ? MvShape{2, 8, std::min(group_splits(n), most), 1} : MvShape{2, 4, std::min(8, most), 1};
    const int rt = n < 3072 || (f64 && ng >= 3) ? 1 : 2;
    // splits for about 1024 blocks; 8 with two groups of FP64 sums.  FP64 sums
    // take no fewer, and no shape takes more where its partial sums and packed
    // right-hand sides would then outgrow bem_matvec_noalloc's array.
    const int rows = f64 ? 64 : 128, blocks = (n + rows - 1) / rows;
    const int usual = f64 && ng == 2 ? 8 : std::max(1, std::min((1023 + blocks) / blocks, n / 256));
    const int fit = (int)(BEM_NOALLOC_SCRATCH_BYTES / ((f64 ? sizeof(double2) : sizeof(float2)) * 16 * ng * n)) - 1;
    return {rt, 4, wide_splits(n, rt, f64, f64 ? usual : 1, std::min(most, std::max(usual, fit))), 1};
}

// Shapes of the row-block products (in a table row: vector class rt = 1, one
// group of 16 g3 = 2; both values had no meaning of their own before).
constexpr MvShape ROW_VEC{1, 0, 1, 0}, ROW_MFMA{1, 4, 1, 2};
bool row_shape(int ng, const MvShape& c) { return ng == 0 ? c.rt == 1 : ng == 1 && c.g3 == 2; }

// A system takes the row-block product by itself while its matrix fits the 256
// MiB Infinity Cache (n <= 4096 in FP64, 5792 in FP32) and it has up to 16
// right-hand sides.  Both ways timed through bem_matvec, us (split / row-block;
// 10 is what the call costs the host), 1, 3 and 16 right-hand sides, FP64:
//   n  512  12.6 / 10.2   12.5 / 10.2   15.0 / 10.8
//   n 1554  18.3 / 10.1   27.2 / 14.2   28.4 / 20.7
//   n 2674  29.6 / 19.1   37.5 / 23.1   38.2 / 30.6
//   n 4096  69.5 / 40.0   64.1 / (X does not fit)  58.1 / 47.9
//   n 5400  88.9 / 103    110 / -       114 / 141
// FP32: n 2674  22.7 / 12.3, 43.3 / 15.8, 29.6 / 22.7; n 5400  53.5 / 41.2,
// 75.6 / 63.9, 73.5 / 75.3; n 6800  70.3 / 69.1, 110 / -, 89 / 126.
bool row_default(int types, int ng, int n)
{
    return ng <= 1 && (size_t)n * n * (types & 2 ? sizeof(double2) : sizeof(float2)) <= ((size_t)256 << 20);
}

// The built-in shapes of a class (vector: ng = 0): split over columns, and the
// one it takes by itself.
MvShape split_shape(int types, int ng, int n)
{
    return ng == 0 ? MvShape{0, 0, matvec_splits_valu(n), 0} : mfma_default(n, ng, types & 1);
}
MvShape default_shape(int types, int ng, int n)
{
    if (row_default(types, ng, n)) return ng == 0 ? ROW_VEC : ROW_MFMA;
    return split_shape(types, ng, n);
}

bool shape_valid(int ng, const MvShape& c)
{
    if (ng == 0) return c.splits >= 1 && c.splits <= 64;
    const bool ok = ng == 1 ? ((c.rt == 1 || c.rt == 2 || c.rt == 4) && (c.u == 2 || c.u == 4 || c.u == 8))
                            : ((c.rt == 1 || c.rt == 2) && (c.u == 2 || c.u == 4) && c.g3 == 1);
    return ok && c.splits >= 1 && c.splits <= 64;
}

// ---------------------------------------------------------------------------
// Launch-shape table.  A class is (type pair, right-hand-side groups, size
// class): types = 2 [matrix stored in FP64] + [accumulation in FP64]; ng = 0
// for the vector kernel (up to 4 right-hand sides), 1-4 for the matrix-core
// kernel; size class = ceil(log2 n).  bem_tune fills the table; the tuner's
// candidate under test is forced per thread.  Column splits never exceed
// split_cap(n, ng), by which the partial-sum buffer is sized, so buffers sized
// before or after tuning stay valid.
// ---------------------------------------------------------------------------
struct ShapeKey {
    int types, ng, lg;
    bool operator<(const ShapeKey& o) const
    {
        return types != o.types ? types < o.types : (ng != o.ng ? ng < o.ng : lg < o.lg);
    }
};
std::mutex g_tune_mu;
std::map<ShapeKey, MvShape> g_tuned;
thread_local const MvShape* g_forced = nullptr;

int size_class(int n)
{
    int lg = 0;
    while (lg < 31 && (1 << lg) < n) ++lg;
    return lg;
}

int split_cap(int n, int ng) { return ng == 0 ? matvec_splits_valu(n) : split_limit(n, ng); }

// Environment overrides of the launch shape (manual tuning): BEM_MV_CFG for
// one group of 16 right-hand sides, BEM_MV_CFG_WIDE for 2-4 groups,
// "rt,u,splits[,g3]".
bool env_shape(int ng, MvShape& out)
{
    const char* e = getenv(ng == 1 ? "BEM_MV_CFG" : "BEM_MV_CFG_WIDE");
    if (!e) return false;
    MvShape t{0, 0, 0, 1};
    const int got = sscanf(e, "%d,%d,%d,%d", &t.rt, &t.u, &t.splits, &t.g3);
    if (ng > 1) t.g3 = 1;
    t.g3 = t.g3 != 0;
    if (got < 3 || !shape_valid(ng, t)) return false;
    out = t;
    return true;
}

}  // namespace

// A frozen source of shapes: the tuned table and the environment overrides.
struct ShapeSnapshot {
    std::map<ShapeKey, MvShape> table;
    bool have_env[2] = {false, false};  // [0]: one group, [1]: 2-4 groups
    MvShape env[2] = {};
};

namespace {

// The shape a product of this class runs with, from a snapshot (or the live
// table and environment when snap is null): an environment override, else the
// tuned table, else the default; splits clamped to split_cap.
MvShape shape_from(const ShapeSnapshot* snap, int types, int ng, int n)
{
    MvShape c = default_shape(types, ng, n);
    bool have = false;
    if (ng > 0) {
        MvShape t{};
        if (snap ? snap->have_env[ng > 1] : env_shape(ng, t)) {
            c = snap ? snap->env[ng > 1] : t;
            have = true;
        }
    }
    if (!have) {
        const ShapeKey key{types, ng, size_class(n)};
        if (snap) {
            auto it = snap->table.find(key);
            if (it != snap->table.end()) c = it->second;
        } else {
            std::lock_guard<std::mutex> lk(g_tune_mu);
            auto it = g_tuned.find(key);
            if (it != g_tuned.end()) c = it->second;
        }
    }
    c.splits = std::max(1, std::min({c.splits, split_cap(n, ng), std::max(1, n / 64)}));
    return c;
}

// The shape a launch uses: the tuner's forced candidate (this thread), else the
// problem's resolved shapes, else the live table (callers without a problem).
MvShape pick_shape(const MvShapes* shapes, int types, int ng, int n)
{
    if (g_forced && shape_valid(ng, *g_forced)) {
        MvShape c = *g_forced;
        c.splits = std::max(1, std::min({c.splits, split_cap(n, ng), std::max(1, n / 64)}));
        return c;
    }
    if (shapes) return shapes->s[types][ng];
    return shape_from(nullptr, types, ng, n);
}


template <class TA, class T, class V2>
void launch_mfma_variant(const MvShape& c, int ng, dim3 grid, hipStream_t s, const TA* A, size_t lda, int n,
                         const V2* xt, int nr, V2* part, int cps)
{
#define BEM_MV_LAUNCH(RT_, U_, G3_, NG_) \
    hipLaunchKernelGGL((k_matvec_mfma<TA, T, RT_, U_, G3_, NG_>), grid, dim3(BS), 0, s, A, lda, n, xt, nr, part, cps)
#define BEM_MV_CASE(RT_, U_)                         \
    if (c.rt == RT_ && c.u == U_) {                  \
        if (c.g3)                                    \
            BEM_MV_LAUNCH(RT_, U_, true, 1);         \
        else                                         \
            BEM_MV_LAUNCH(RT_, U_, false, 1);        \
        return;                                      \
    }
#define BEM_MV_WIDE(RT_, U_)                                  \
    if (c.rt == RT_ && c.u == U_) {                           \
        if (ng == 2)                                          \
            BEM_MV_LAUNCH(RT_, U_, true, 2);                  \
        else if (ng == 3)                                     \
            BEM_MV_LAUNCH(RT_, U_, true, 3);                  \
        else                                                  \
            BEM_MV_LAUNCH(RT_, U_, true, 4);                  \
        return;                                               \
    }
    if (ng == 1) {
        BEM_MV_CASE(1, 2)
        BEM_MV_CASE(1, 4)
        BEM_MV_CASE(1, 8)
        BEM_MV_CASE(2, 2)
        BEM_MV_CASE(2, 4)
        BEM_MV_CASE(2, 8)
        BEM_MV_CASE(4, 2)
        BEM_MV_CASE(4, 4)
        BEM_MV_CASE(4, 8)
    } else {
        BEM_MV_WIDE(1, 2)
        BEM_MV_WIDE(1, 4)
        BEM_MV_WIDE(2, 2)
        BEM_MV_WIDE(2, 4)
    }
#undef BEM_MV_WIDE
#undef BEM_MV_CASE
#undef BEM_MV_LAUNCH
}

template <class TA, class TX, class ACC, class TY>
hipError_t matvec_any(const TA* A, size_t lda, int n, const TX* X, size_t ldx, int nrhs, TY* Y, size_t ldy,
                      ACC* part, const double2* B, size_t ldb, hipStream_t s, const KernelHook* hook,
                      const MvShapes* shapes)
{
    using S = decltype(ACC{}.x);
    constexpr int types = (sizeof(TA) == 16 ? 2 : 0) + (sizeof(S) == 8 ? 1 : 0);
    const int rowblocks = (n + 64 * MV_WAVES - 1) / (64 * MV_WAVES);
    const int kind = B ? KIND_RESIDUAL : KIND_MATVEC;
    const bool in_place = blocks_overlap(X, ldx * sizeof(TX), Y, ldy * sizeof(TY), nrhs);
    for (int r0 = 0; r0 < nrhs; r0 += MFMA_MAX_RHS) {
        const int nr = std::min(MFMA_MAX_RHS, nrhs - r0);
        const TX* Xg = X + (size_t)r0 * ldx;
        const double2* Bg = B ? B + (size_t)r0 * ldb : nullptr;
        const int ng = nr > 4 ? (nr + 15) / 16 : 0;
        const MvShape picked = pick_shape(shapes, types, ng, n);
        const bool row = row_shape(ng, picked) && !in_place && row_fits(n, nr, sizeof(ACC));
        const MvShape cfg = row || !row_shape(ng, picked) ? picked : split_shape(types, ng, n);
        if (row) {
            const RowOut<TY, double2> o{Y + (size_t)r0 * ldy, ldy, Bg, ldb, nullptr, 0, nullptr, 0, nullptr, nullptr};
            hook_call(hook, kind, 0, s);
            if (B)
                launch_rowblock<TA, TX, ACC, false, ROW_RESIDUAL>(A, lda, n, Xg, ldx, nr, o, s);
            else
                launch_rowblock<TA, TX, ACC, false, ROW_PRODUCT>(A, lda, n, Xg, ldx, nr, o, s);
            hook_call(hook, kind, 1, s);
            continue;
        }
        if (ng > 0) {
            // pack X right-hand-side fastest into the tail of the partial buffer
            const int ms = cfg.splits;
            const int mcps = ((n + ms - 1) / ms + 31) / 32 * 32;
            ACC* xt = part + (size_t)ms * nr * n;
            hipLaunchKernelGGL((k_pack_xt<TX, ACC>), dim3(((size_t)n * 16 * ng + BS - 1) / BS), dim3(BS), 0, s, Xg,
                               ldx, n, nr, 16 * ng, xt);
            hook_call(hook, kind, 0, s);
            const int rows_per_block = 16 * cfg.rt * MV_WAVES;
            launch_mfma_variant<TA, S, ACC>(cfg, ng, dim3((n + rows_per_block - 1) / rows_per_block, ms), s, A, lda,
                                            n, xt, nr, part, mcps);
            hook_call(hook, kind, 1, s);
            hipLaunchKernelGGL((k_matvec_reduce<ACC, TY>), dim3((n + BS - 1) / BS, nr), dim3(BS), 0, s, part, ms, n,
                               nr, Y + (size_t)r0 * ldy, ldy, Bg, ldb);
            continue;
        }
        const int splits = cfg.splits;
        const int cps = (n + splits - 1) / splits;
        dim3 grid(rowblocks, splits);
        hook_call(hook, kind, 0, s);
        if (nr == 1)
            hipLaunchKernelGGL((k_matvec<1, TA, TX, ACC>), grid, dim3(BS), 0, s, A, lda, n, Xg, ldx, nr, part, cps);
        else if (nr == 2)
            hipLaunchKernelGGL((k_matvec<2, TA, TX, ACC>), grid, dim3(BS), 0, s, A, lda, n, Xg, ldx, nr, part, cps);
        else
            hipLaunchKernelGGL((k_matvec<4, TA, TX, ACC>), grid, dim3(BS), 0, s, A, lda, n, Xg, ldx, nr, part, cps);
        hook_call(hook, kind, 1, s);
        hipLaunchKernelGGL((k_matvec_reduce<ACC, TY>), dim3((n + BS - 1) / BS, nr), dim3(BS), 0, s, part, splits, n,
                           nr, Y + (size_t)r0 * ldy, ldy, Bg, ldb);
    }
    return hipGetLastError();
}

__device__ __forceinline__ void st_basis(double2* p, double2 v) { *p = v; }
__device__ __forceinline__ void st_basis(float2* p, double2 v) { *p = make_float2((float)v.x, (float)v.y); }

// The split reduction of a Krylov step's product whose inputs were w of the
// previous step, not yet divided by |w|: Y = (sum of the split partial sums,
// in split order) / |w| = A v_j, and before Y overwrites w (Y is the step's w
// buffer): v_j = w / |w| into the basis for active columns, |w| into hnorm,
// and the stopping marks of the previous step cleared (what the
// normalisation kernel does otherwise).
template <class ACC, class TV>
__global__ void k_step_reduce(const ACC* __restrict__ part, int splits, int n, int nrhs, double2* __restrict__ Y,
                              size_t ldy, const double* __restrict__ nrm, int nu, TV* __restrict__ V, size_t ldv,
                              double* __restrict__ hnorm, int* __restrict__ active)
{
    __shared__ double inv_s;
    const int r = blockIdx.y;
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    const int act = active[r];
    // this thread's loads first (they do not depend on |w|), then |w|
    double sr = 0.0, si = 0.0;
    double2 w = make_double2(0.0, 0.0);
    double2* y = Y + (size_t)r * ldy + row;
    if (row < n) {
        for (int sp = 0; sp < splits; ++sp) {
            const ACC v = part[((size_t)sp * nrhs + r) * n + row];
            sr += v.x;
            si += v.y;
        }
        w = *y;
    }
    if (threadIdx.x < 64) {
        const double beta = dev::step_beta(nrm + (size_t)r * nu, nu);
        if (threadIdx.x == 0) {
            inv_s = dev::inv_beta(beta);
            if (blockIdx.x == 0 && act == 1) hnorm[r] = beta;
        }
    }
    __syncthreads();
    // every block of a marked column skips it, whether it reads the mark or the zero
    if (blockIdx.x == 0 && threadIdx.x == 0 && act == dev::STOPPING) active[r] = 0;
    if (row >= n) return;
    const double inv = inv_s;
    if (act == 1) st_basis(V + (size_t)r * ldv + row, make_double2(w.x * inv, w.y * inv));
    *y = make_double2(sr * inv, si * inv);
}

// Products of the Krylov steps whose inputs the caller has packed at part +
// xt_offset: the row-block product, or (5-64 right-hand sides) the matrix-core
// kernel and the split reduction (with sn: inputs not yet normalised, see
// k_step_reduce).
template <class TA, class ACC>
hipError_t product_packed(const ProductPlan& pl, const TA* A, size_t lda, int n, int nr, ACC* part, double2* Y,
                          size_t ldy, const StepNorm* sn, hipStream_t s, const KernelHook* hook)
{
    using S = decltype(ACC{}.x);
    if (pl.row) {
        const ACC* xt = part + pl.xt_offset;
        hook_call(hook, KIND_MATVEC, 0, s);
        if (!sn)
            launch_rowblock<TA, ACC, ACC, true, ROW_PRODUCT>(
                A, lda, n, xt, 0, nr, RowOut<double2, double2>{Y, ldy, nullptr, 0, nullptr, 0, nullptr, 0, nullptr, nullptr}, s);
        else if (sn->v32)
            launch_rowblock<TA, ACC, ACC, true, ROW_STEP>(
                A, lda, n, xt, 0, nr,
                RowOut<double2, float2>{Y, ldy, nullptr, 0, sn->norm_part, sn->nu, static_cast<float2*>(sn->V), sn->ldv,
                                        sn->hnorm, sn->active}, s);
        else
            launch_rowblock<TA, ACC, ACC, true, ROW_STEP>(
                A, lda, n, xt, 0, nr,
                RowOut<double2, double2>{Y, ldy, nullptr, 0, sn->norm_part, sn->nu, static_cast<double2*>(sn->V),
                                         sn->ldv, sn->hnorm, sn->active}, s);
        hook_call(hook, KIND_MATVEC, 1, s);
        return hipGetLastError();
    }
    const int rows_per_block = 16 * pl.shape.rt * MV_WAVES;
    const int mcps = ((n + pl.splits - 1) / pl.splits + 31) / 32 * 32;
    hook_call(hook, KIND_MATVEC, 0, s);
    launch_mfma_variant<TA, S, ACC>(pl.shape, pl.ng, dim3((n + rows_per_block - 1) / rows_per_block, pl.splits), s, A,
                                    lda, n, part + pl.xt_offset, nr, part, mcps);
    hook_call(hook, KIND_MATVEC, 1, s);
    const dim3 grid((n + BS - 1) / BS, nr);
    if (!sn)
        hipLaunchKernelGGL((k_matvec_reduce<ACC, double2>), grid, dim3(BS), 0, s, part, pl.splits, n, nr, Y, ldy,
                           nullptr, 0);
    else if (sn->v32)
        hipLaunchKernelGGL((k_step_reduce<ACC, float2>), grid, dim3(BS), 0, s, part, pl.splits, n, nr, Y, ldy,
                           sn->norm_part, sn->nu, static_cast<float2*>(sn->V), sn->ldv, sn->hnorm, sn->active);
    else
        hipLaunchKernelGGL((k_step_reduce<ACC, double2>), grid, dim3(BS), 0, s, part, pl.splits, n, nr, Y, ldy,
                           sn->norm_part, sn->nu, static_cast<double2*>(sn->V), sn->ldv, sn->hnorm, sn->active);
    return hipGetLastError();
}

}  // namespace

ProductPlan product_plan(const MvShapes* shapes, int types, int n, int nr)
{
    ProductPlan pl{};
    pl.ng = nr > 4 ? (nr + 15) / 16 : 0;
    pl.shape = pick_shape(shapes, types, pl.ng, n);
    pl.row = row_shape(pl.ng, pl.shape) && row_fits(n, nr, types & 1 ? sizeof(double2) : sizeof(float2));
    if (!pl.row && row_shape(pl.ng, pl.shape)) pl.shape = split_shape(types, pl.ng, n);
    pl.packed = pl.row || pl.ng > 0;
    pl.splits = pl.shape.splits;
    pl.xt_offset = pl.packed && !pl.row ? (size_t)pl.splits * nr * n : 0;
    pl.xw = pl.ng > 0 ? 16 * pl.ng : pl.row ? nr : 0;
    return pl;
}

hipError_t launch_product_packed_f64(const ProductPlan& pl, const double2* A, size_t lda, int n, int nr,
                                     double2* part, double2* Y, size_t ldy, const StepNorm* sn, hipStream_t s,
                                     const KernelHook* hook)
{
    return product_packed<double2, double2>(pl, A, lda, n, nr, part, Y, ldy, sn, s, hook);
}

hipError_t launch_product_packed_f32(const ProductPlan& pl, const float2* A, size_t lda, int n, int nr,
                                     float2* part, double2* Y, size_t ldy, const StepNorm* sn, hipStream_t s,
                                     const KernelHook* hook)
{
    return product_packed<float2, float2>(pl, A, lda, n, nr, part, Y, ldy, sn, s, hook);
}

int matvec_splits_valu(int n)
{
    // enough column splits that the grid holds >= ~1024 blocks of 4 waves,
    // but never fewer than 64 columns per split
    const int rowblocks = (n + 64 * MV_WAVES - 1) / (64 * MV_WAVES);
    int s = (1024 + rowblocks - 1) / rowblocks;
    const int maxs = std::max(1, n / 64);
    if (s > maxs) s = maxs;
    if (s > 64) s = 64;
    return std::max(1, s);
}

// Partial-sum buffer of a product with nrhs right-hand sides, in complex
// values of the accumulation type: the column-split partial sums of the
// largest chunk plus the packed copy of X (matrix-core path).  Sized for the
// FP64 shape; an FP32 product uses the same shape with half-size values.
size_t matvec_part_elems(int n, int nrhs)
{
    const int nr = std::min(nrhs, MFMA_MAX_RHS);
    size_t e = (size_t)split_cap(n, 0) * std::min(nr, 4);
    if (nr > 4) {
        const int ng = (nr + 15) / 16;
        e = std::max(e, (size_t)split_cap(n, ng) * nr + 16 * ng);
    }
    return e * (size_t)n;
}

bool blocks_overlap(const void* X, size_t xcol, const void* Y, size_t ycol, int nrhs)
{
    const char *x = static_cast<const char*>(X), *y = static_cast<const char*>(Y);
    return x < y + ycol * nrhs && y < x + xcol * nrhs;
}

size_t matvec_part_elems_shaped(const MvShapes& sh, int types, int n, int nrhs, bool in_place)
{
    size_t e = 0;
    for (int r0 = 0; r0 < nrhs; r0 += MFMA_MAX_RHS) {
        const int nr = std::min(MFMA_MAX_RHS, nrhs - r0);
        const int ng = nr > 4 ? (nr + 15) / 16 : 0;
        const bool row = row_shape(ng, sh.s[types][ng]);
        if (row && !in_place && row_fits(n, nr, types & 1 ? sizeof(double2) : sizeof(float2)))
            continue;  // neither partial sums nor a packed copy
        const size_t c = (size_t)(row ? split_shape(types, ng, n) : sh.s[types][ng]).splits * nr + (ng ? 16 * ng : 0);
        e = std::max(e, c);
    }
    return e * (size_t)n;
}

hipError_t launch_matvec_f64(const double2* A, size_t lda, int n, const double2* X, size_t ldx, int nrhs,
                             double2* Y, size_t ldy, double2* partial, hipStream_t s, const KernelHook* hook,
                             const MvShapes* shapes)
{
    return matvec_any<double2, double2, double2, double2>(A, lda, n, X, ldx, nrhs, Y, ldy, partial, nullptr, 0, s,
                                                          hook, shapes);
}

hipError_t launch_matvec_f32(const float2* A, size_t lda, int n, const float2* X, size_t ldx, int nrhs, float2* Y,
                             size_t ldy, float2* partial, hipStream_t s, const KernelHook* hook,
                             const MvShapes* shapes)
{
    return matvec_any<float2, float2, float2, float2>(A, lda, n, X, ldx, nrhs, Y, ldy, partial, nullptr, 0, s, hook,
                                                      shapes);
}

hipError_t launch_matvec_f32x64(const float2* A, size_t lda, int n, const double2* X, size_t ldx, int nrhs,
                                double2* Y, size_t ldy, float2* partial, hipStream_t s, const KernelHook* hook,
                             const MvShapes* shapes)
{
    return matvec_any<float2, double2, float2, double2>(A, lda, n, X, ldx, nrhs, Y, ldy, partial, nullptr, 0, s, hook,
                                                        shapes);
}

hipError_t launch_matvec_f32v(const float2* A, size_t lda, int n, const float2* X, size_t ldx, int nrhs,
                              double2* Y, size_t ldy, float2* partial, hipStream_t s, const KernelHook* hook,
                             const MvShapes* shapes)
{
    return matvec_any<float2, float2, float2, double2>(A, lda, n, X, ldx, nrhs, Y, ldy, partial, nullptr, 0, s, hook,
                                                       shapes);
}

hipError_t launch_residual_f64(const double2* A, size_t lda, int n, const double2* X, size_t ldx, int nrhs,
                              const double2* B, size_t ldb, double2* R, size_t ldr, double2* partial, hipStream_t s,
                              const KernelHook* hook, const MvShapes* shapes)
{
    return matvec_any<double2, double2, double2, double2>(A, lda, n, X, ldx, nrhs, R, ldr, partial, B, ldb, s, hook,
                                                          shapes);
}

hipError_t launch_residual_f32A(const float2* A, size_t lda, int n, const double2* X, size_t ldx, int nrhs,
                                const double2* B, size_t ldb, double2* R, size_t ldr, double2* partial,
                                hipStream_t s, const KernelHook* hook,
                                const MvShapes* shapes)
{
    return matvec_any<float2, double2, double2, double2>(A, lda, n, X, ldx, nrhs, R, ldr, partial, B, ldb, s, hook,
                                                         shapes);
}


// ---------------------------------------------------------------------------
// Tuning table access (bem_tune and its export / import).
// ---------------------------------------------------------------------------
void force_shape(const MvShape* s) { g_forced = s; }

MvShape current_shape(int types, int ng, int n) { return shape_from(nullptr, types, ng, n); }

std::shared_ptr<const ShapeSnapshot> snapshot_shapes()
{
    auto snap = std::make_shared<ShapeSnapshot>();
    for (int w = 0; w < 2; ++w) snap->have_env[w] = env_shape(w ? 2 : 1, snap->env[w]);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    snap->table = g_tuned;
    return snap;
}

void resolve_shapes(const ShapeSnapshot* snap, int n, MvShapes& out)
{
    for (int t = 0; t < 4; ++t)
        for (int ng = 0; ng <= 4; ++ng) out.s[t][ng] = shape_from(snap, t, ng, n);
}

std::vector<MvShape> candidate_shapes(int types, int ng, int n)
{
    std::vector<MvShape> out;
    const int cap = split_cap(n, ng);
    std::vector<int> splits;
    for (int s = cap; s >= 1; s /= 2) splits.push_back(s);
    const MvShape d = default_shape(types, ng, n);
    out.push_back(d);  // the default first
    if (ng <= 1 && !row_shape(ng, d)) out.push_back(ng == 0 ? ROW_VEC : ROW_MFMA);
    if (ng == 0) {
        for (int s : splits)
            if (row_shape(0, d) || s != d.splits) out.push_back(MvShape{0, 0, s, 0});
        return out;
    }
    const int rts[] = {1, 2, 4}, us[] = {2, 4, 8};
    for (int rt : rts)
        for (int u : us)
            for (int g3 = (ng == 1 ? 0 : 1); g3 <= 1; ++g3)
                for (int s : splits) {
                    const MvShape c{rt, u, s, g3};
                    if (!shape_valid(ng, c)) continue;
                    if (c.rt == d.rt && c.u == d.u && c.g3 == d.g3 && c.splits == d.splits) continue;
                    out.push_back(c);
                }
    return out;
}

void set_tuned_shape(int types, int ng, int n, const MvShape& c)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned[ShapeKey{types, ng, size_class(n)}] = c;
}

void clear_tuned_shapes()
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned.clear();
}

std::string export_tuned_shapes()
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    std::ostringstream o;
    o << "# bem product launch shapes: types ng log2n rt u splits g3\n";
    for (const auto& kv : g_tuned)
        o << kv.first.types << ' ' << kv.first.ng << ' ' << kv.first.lg << ' ' << kv.second.rt << ' ' << kv.second.u
          << ' ' << kv.second.splits << ' ' << kv.second.g3 << '\n';
    return o.str();
}

bool import_tuned_shapes(const char* text)
{
    std::map<ShapeKey, MvShape> add;
    std::istringstream in(text ? text : "");
    std::string line;
    while (std::getline(in, line)) {
        if (line.empty() || line[0] == '#') continue;
        std::istringstream l(line);
        ShapeKey k{};
        MvShape c{};
        if (!(l >> k.types >> k.ng >> k.lg >> c.rt >> c.u >> c.splits >> c.g3)) return false;
        std::string rest;
        if (l >> rest) return false;
        if (k.types < 0 || k.types > 3 || k.types == 2 || k.ng < 0 || k.ng > 4 || k.lg < 0 || k.lg > 31) return false;
        if (!shape_valid(k.ng, c)) return false;
        add[k] = c;
    }
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (const auto& kv : add) g_tuned[kv.first] = kv.second;
    return true;
}

}  // namespace bemk
