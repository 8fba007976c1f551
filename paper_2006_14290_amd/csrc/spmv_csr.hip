// spmv_csr.hip -- load-balanced CSR sparse matrix-vector product for gfx950.
//
// y = alpha * A x + beta * y over the Csr format (Section 1 of the paper
// lists it among the library's formats; Section 4 measures its SpMV).
//
// Matrices of known, similar row lengths take the staged-rows kernel
// (spmv_csr_stage.hpp); the rest of this comment describes the tile kernel.
//
// Work split: the nonzeros are cut into tiles of kTile entries; tile k owns
// every row that STARTS inside [k*kTile, (k+1)*kTile) and processes the whole
// nonzero range of those rows. Each work-group finds its rows with two
// wavefront-cooperative 64-ary searches of the row pointer, streams the
// range in passes of kTile products staged in LDS (coalesced, non-temporal
// loads of values and column indices; gathers of x through the caches), and
// reduces the rows of a pass with subwarps whose size is chosen from the
// number of rows in the pass (Section 3.3's subwarp model: many short rows ->
// small subwarps, one long row -> a whole wavefront). A row longer than a pass
// carries its partial sum in LDS to the next pass. Every row is written once
// by its owner: no atomics, and the summation order is fixed, so results are
// bitwise reproducible.
//
// Bytes moved (the roofline unit): nnz*(sv+4) + (nrows+1)*4 + ncols*sx +
// nrows*sx (+ nrows*sx when beta != 0).
#include "common.hpp"
#include "krylov.hpp"
#include "spmv_csr.hpp"
#include "spmv_csr_stage.hpp"
#include "spmv_csr_tile.hpp"
#include "wave.hpp"

namespace spx {

// One work-group per tile (XCD-remapped block id); see csr_tile. With a
// solver state, a set flag skips the launch.
template <typename V, typename X, int kEpi, int kThreads, int kTile, int kVec, bool kLate>
__global__ __launch_bounds__(kThreads) void csr_spmv_kernel(
    int32_t nrows, int64_t nnz, int64_t ntiles, int64_t grid_padded, const int32_t *__restrict__ rowptr,
    const int32_t *__restrict__ col, const V *__restrict__ val, const X *__restrict__ x, X *__restrict__ y,
    X alpha, X beta, const X *__restrict__ dot_with, X *__restrict__ dot_partials, const int32_t *__restrict__ part,
    KState *__restrict__ st, int op)
{
    if (st != nullptr && st->flag != kRunning) return;
    const int64_t k = xcd_remap(blockIdx.x, grid_padded);
    if (k >= ntiles) return;
    __shared__ __align__(16) unsigned char s_raw[csr_tile_lds<V, X, kTile, kLate>()];
    csr_tile<V, X, kEpi, kThreads, kTile, kVec, kLate>(s_raw, k, nrows, nnz, ntiles, rowptr, col, val, x, y, alpha,
                                                       beta, dot_with, dot_partials, part);
}

// Row-per-subwarp CSR product for short, regular rows (the "classical"
// strategy: a subwarp of kSub lanes per row, kSub the power of two at or
// above the mean row length). A block takes kRowU * kRowThreads / kSub
// consecutive rows; at step u the subwarps of a wavefront hold adjacent rows,
// so every load instruction reads one contiguous stretch of col / val. The
// first kSub entries of all kRowU rows are loaded before the first gather;
// longer rows continue in a loop. Rows are reduced with DPP (fixed order).
// A block does this `steps` times, over the rows that follow: once, as what
// bounds it is the chain of its three dependent loads (row pointer, column, x)
// and every further step adds the whole chain again (4,096 rows in 4 blocks of
// eight steps: 13.6 us; in 32 blocks of one: 3.7); eight times where the sums'
// order is to be kept (row_steps).
template <typename V, typename X, int kEpi, int kSub>
__global__ __launch_bounds__(kRowThreads) void csr_rows_kernel(
    int32_t nrows, int64_t nblocks, int64_t grid_padded, const int32_t *__restrict__ rowptr,
    const int32_t *__restrict__ col, const V *__restrict__ val, const X *__restrict__ x, X *__restrict__ y, X alpha,
    X beta, const X *__restrict__ dot_with, X *__restrict__ dot_partials, KState *__restrict__ st, int steps)
{
    if (st != nullptr && st->flag != kRunning) return;
    constexpr int kSubs = kRowThreads / kSub;
    constexpr int64_t kStep = (int64_t)kSubs * kRowU;  // rows per block iteration
    const int64_t blk = xcd_remap(blockIdx.x, grid_padded);
    if (blk >= nblocks) return;
    const int tid = threadIdx.x, sw = tid / kSub, sl = tid % kSub;
    X d1 = X(0), d2 = X(0);
    for (int it = 0; it < steps; ++it) {
        const int64_t base = (blk * steps + it) * kStep + sw;
        if (base - sw >= nrows) break;  // uniform across the block
        int32_t a[kRowU], b[kRowU], c[kRowU];
        V v[kRowU];
#pragma unroll
        for (int u = 0; u < kRowU; ++u) {
            const int64_t row = base + (int64_t)u * kSubs;
            a[u] = 0;
            b[u] = 0;
            if (row < nrows) {
                a[u] = rowptr[row];
                b[u] = rowptr[row + 1];
            }
        }
#pragma unroll
        for (int u = 0; u < kRowU; ++u) {
            const int32_t k = a[u] + sl;
            c[u] = -1;
            v[u] = V(0);
            if (k < b[u]) {
                c[u] = ld_stream(col + k);
                v[u] = ld_stream(val + k);
            }
        }
        X sum[kRowU];
#pragma unroll
        for (int u = 0; u < kRowU; ++u) sum[u] = c[u] >= 0 ? widen(v[u]) * x[c[u]] : X(0);
#pragma unroll
        for (int u = 0; u < kRowU; ++u)
            for (int32_t k = a[u] + sl + kSub; k < b[u]; k += kSub)
                sum[u] += widen(ld_stream(val + k)) * x[ld_stream(col + k)];
#pragma unroll
        for (int u = 0; u < kRowU; ++u) {
            const X t = subwave_sum<kSub>(sum[u]);
            const int64_t row = base + (int64_t)u * kSubs;
            if (sl == 0 && row < nrows) {
                X out = alpha * t;
                if (beta != X(0)) out += beta * y[row];
                y[row] = out;
                if constexpr (kEpi >= 1) d1 += out * dot_with[row];
                if constexpr (kEpi >= 2) d2 += out * out;
            }
        }
    }
    if constexpr (kEpi > 0) {
        __shared__ X s_red[kRowThreads / kWave];
        X vv[kEpi];
        vv[0] = block_sum<X, kRowThreads>(d1, s_red);
        if constexpr (kEpi >= 2) vv[kEpi - 1] = block_sum<X, kRowThreads>(d2, s_red);
        write_partials<X, kEpi>(vv, dot_partials, nblocks, blk);
    }
}

// One wavefront per tile boundary k in [0, ntiles]: the first row starting
// at or after k*kCsrTile (nrows for the final boundary) and its offset.
__global__ __launch_bounds__(256) void csr_partition_kernel(int32_t nrows, int64_t nnz, int64_t ntiles,
                                                           const int32_t *__restrict__ rowptr,
                                                           int32_t *__restrict__ part)
{
    const int64_t k = (int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
    if (k > ntiles) return;
    int32_t v = (int32_t)nnz;
    int64_t r = nrows;
    if (k < ntiles) r = lower_bound_wave(rowptr, 0, nrows, k * kCsrTile, &v);
    if (lane_id() == 0) {
        part[2 * k] = (int32_t)r;
        part[2 * k + 1] = v;
    }
}

spx_status csr_partition_launch(const spx_matrix &A, int32_t *part, hipStream_t stream)
{
    const int64_t ntiles = csr_tiles(A.nnz);
    csr_partition_kernel<<<(unsigned)ceil_div(ntiles + 1, 256 / kWave), 256, 0, stream>>>(A.nrows, A.nnz, ntiles,
                                                                                          A.rowptr, part);
    SPX_LAUNCHED();
    return SPX_OK;
}

// The staged-rows kernel (spmv_csr_stage.hpp) for A: the row length its
// unrolled part holds (8, 16, 32, 64 or 128 entries), or 0 when A takes
// another kernel. Rows must be known to fit that length and fill at least
// half of it on average: a random matrix of 5 to 45 entries per row (mean
// 16.5) ran 2 to 6 % slower than on the tile kernel with half-empty stages,
// the stencils 5 to 60 % faster. Fewer than kStageMinNnz entries (and arrays
// that 16-byte copies cannot read) keep the tile kernel.
static int stage_len(const spx_matrix &A)
{
    if (A.csr_cb_tiles == kCsrNoStage) return 0;
    if (A.max_row_len <= 0 || A.nrows <= 0 || A.nnz < kStageMinNnz || A.nnz > INT32_MAX - kStageMinNnz) return 0;
    if (((reinterpret_cast<uintptr_t>(A.colidx) | reinterpret_cast<uintptr_t>(A.vals)) & 15) != 0) return 0;
    for (int len = 8; len <= 128; len *= 2)
        if (A.max_row_len <= len) return 2 * A.nnz >= (int64_t)len * A.nrows ? len : 0;
    return 0;
}

int csr_rows_sub(const spx_matrix &A)
{
    // measured on gfx950 against the tile kernel, 5 to 45 random entries per
    // row: 3,000 rows 3.8 / 3.5 us, 20,000 rows 5.1 / 6.1, 60,000 rows 9.8 /
    // 8.6. Below kStageMinNnz entries (1,089 rows of 5) 3.2 / 5.2.
    if (stage_len(A) > 0) return 0;
    const int32_t most = A.csr_cb_tiles == kCsrNoStage ? 2 * kRowMaxRows : kRowMaxRows;
    if (A.nrows <= 0 || A.nrows > most || A.max_row_len <= 0 || A.nnz <= 0) return 0;
    const int64_t mean = ceil_div(A.nnz, A.nrows);
    int sub = 4;
    while (sub < 64 && sub < mean) sub <<= 1;
    return A.max_row_len <= 2 * sub ? sub : 0;
}

// Rows per block, work-groups per CU and grid of the staged-rows kernel.
// float64 stages 512 entries per wavefront (6 KB) with three work-groups per
// CU resident, narrower values 1024 (6 to 8 KB) with four: 27-point float64
// 70.2 / 63.3 / 66.9 us with two / three / four, float32 42.6 / 39.7 / 39.4.
static int stage_rows(const spx_matrix &A, int len) { return (A.val_type == SPX_F64 ? 512 : 1024) / len; }

static int64_t stage_grid(const spx_matrix &A, int len)
{
    const int64_t wgs = ceil_div(ceil_div(A.nrows, stage_rows(A, len)), kStageWaves);
    const int64_t most = 256 * (A.val_type == SPX_F64 ? 3 : 4);
    return pad_to_xcds(wgs < most ? wgs : most);
}

template <typename V, typename X, int kEpi>
static void stage_launch(const spx_matrix &A, int len, const X *x, X *y, X alpha, X beta, const X *dot_with,
                         X *dot_partials, hipStream_t stream, KState *st)
{
    const int32_t nblk = (int32_t)ceil_div(A.nrows, stage_rows(A, len));
    const int32_t nnz8 = (int32_t)(A.nnz & ~(int64_t)7);
    const unsigned grid = (unsigned)stage_grid(A, len);
#define SPX_STAGE(SIZE, ROWS, LEN, CAP)                                                                             \
    csr_stage_kernel<V, X, kEpi, SIZE, ROWS, LEN, CAP><<<grid, kStageWaves * kWave, 0, stream>>>(                   \
        A.nrows, nnz8, nblk, A.rowptr, A.colidx, static_cast<const V *>(A.vals), x, y, alpha, beta, dot_with,       \
        dot_partials, st)
    if constexpr (sizeof(V) == 8) {
        switch (len) {
        case 8: SPX_STAGE(1, 1, 8, 512); break;
        case 16: SPX_STAGE(2, 1, 8, 512); break;
        case 32: SPX_STAGE(4, 1, 8, 512); break;
        case 64: SPX_STAGE(8, 1, 8, 512); break;
        default: SPX_STAGE(16, 1, 8, 512); break;
        }
    } else {
        switch (len) {
        case 8: SPX_STAGE(1, 2, 8, 1024); break;
        case 16: SPX_STAGE(1, 1, 16, 1024); break;
        case 32: SPX_STAGE(2, 1, 16, 1024); break;
        case 64: SPX_STAGE(4, 1, 16, 1024); break;
        default: SPX_STAGE(8, 1, 16, 1024); break;
        }
    }
#undef SPX_STAGE
}

// Steps of a block of the row-per-subwarp kernel.
static int row_steps(const spx_matrix &A) { return A.nrows > kRowMaxRows ? 8 : 1; }

int64_t csr_dot_parts(const spx_matrix &A)
{
    const int len = stage_len(A);
    if (len > 0) return stage_grid(A, len);
    const int sub = csr_rows_sub(A);
    if (sub == 0) return csr_tiles(A.nnz);
    return ceil_div(A.nrows, (int64_t)(kRowThreads / sub) * kRowU * row_steps(A));
}

template <typename V, typename X>
spx_status csr_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, const X *dot_with,
                           X *dot_partials, hipStream_t stream, int epi, KState *st, int op)
{
    const V *val = static_cast<const V *>(A.vals);
    if (const int len = stage_len(A); len > 0) {
        if (epi == 2) stage_launch<V, X, 2>(A, len, x, y, alpha, beta, dot_with, dot_partials, stream, st);
        else if (epi == 1) stage_launch<V, X, 1>(A, len, x, y, alpha, beta, dot_with, dot_partials, stream, st);
        else stage_launch<V, X, 0>(A, len, x, y, alpha, beta, dot_with, dot_partials, stream, st);
        SPX_LAUNCHED();
        return SPX_OK;
    }
    const int sub = csr_rows_sub(A);
    if (sub > 0) {
        const int64_t nblocks = csr_dot_parts(A);
        const int64_t grid = pad_to_xcds(nblocks);
#define SPX_ROWS_LAUNCH(E, SUB)                                                                                      \
    csr_rows_kernel<V, X, E, SUB><<<(unsigned)grid, kRowThreads, 0, stream>>>(A.nrows, nblocks, grid, A.rowptr,         \
                                                                               A.colidx, val, x, y, alpha, beta,       \
                                                                               dot_with, dot_partials, st, row_steps(A))
#define SPX_ROWS_EPI(SUB)                                                                                            \
    if (epi == 2) SPX_ROWS_LAUNCH(2, SUB);                                                                           \
    else if (epi == 1) SPX_ROWS_LAUNCH(1, SUB);                                                                      \
    else SPX_ROWS_LAUNCH(0, SUB);
        switch (sub) {
        case 4: SPX_ROWS_EPI(4) break;
        case 8: SPX_ROWS_EPI(8) break;
        case 16: SPX_ROWS_EPI(16) break;
        case 32: SPX_ROWS_EPI(32) break;
        default: SPX_ROWS_EPI(64) break;
        }
#undef SPX_ROWS_EPI
#undef SPX_ROWS_LAUNCH
        SPX_LAUNCHED();
        return SPX_OK;
    }
    const int64_t ntiles = csr_tiles(A.nnz);
    const int64_t grid = pad_to_xcds(ntiles);
    // 16-byte value vectors (and matching column vectors) when both arrays
    // are 16-byte aligned, else one entry per load
    constexpr int kVec = 16 / (int)sizeof(V);
    const bool vec = ((reinterpret_cast<uintptr_t>(A.colidx) | reinterpret_cast<uintptr_t>(val)) & 15) == 0;
#define SPX_CSR_LAUNCH(E, VEC)                                                                                   \
    csr_spmv_kernel<V, X, E, kCsrThreads, kCsrTile, VEC, kCsrLateGather><<<(unsigned)grid, kCsrThreads, 0, stream>>>( \
        A.nrows, A.nnz, ntiles, grid, A.rowptr, A.colidx, val, x, y, alpha, beta, dot_with, dot_partials, A.csr_part, \
        st, op)
    if (vec) {
        if (epi == 2) SPX_CSR_LAUNCH(2, kVec);
        else if (epi == 1) SPX_CSR_LAUNCH(1, kVec);
        else SPX_CSR_LAUNCH(0, kVec);
    } else {
        if (epi == 2) SPX_CSR_LAUNCH(2, 1);
        else if (epi == 1) SPX_CSR_LAUNCH(1, 1);
        else SPX_CSR_LAUNCH(0, 1);
    }
#undef SPX_CSR_LAUNCH
    SPX_LAUNCHED();
    return SPX_OK;
}

template spx_status csr_spmv_launch<double, double>(const spx_matrix &, const double *, double *, double, double,
                                                    const double *, double *, hipStream_t, int, KState *, int);
template spx_status csr_spmv_launch<float, float>(const spx_matrix &, const float *, float *, float, float,
                                                  const float *, float *, hipStream_t, int, KState *, int);
template spx_status csr_spmv_launch<_Float16, float>(const spx_matrix &, const float *, float *, float, float,
                                                     const float *, float *, hipStream_t, int, KState *, int);

}  // namespace spx
