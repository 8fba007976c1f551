// spmv_csr.hpp -- launch interface of the CSR product.
#pragma once

#include "common.hpp"

namespace spx {

constexpr int kCsrThreads = 256;  // work-group size (4 wavefronts)
constexpr int kCsrTile = 2048;    // nonzeros per tile and per LDS pass
constexpr int kCsrSlack = 64;     // a pass may run this many entries past its tile
constexpr bool kCsrLateGather = true;  // gather x while reducing rows (see csr_spmv_kernel)
constexpr int kRowThreads = 256;  // row-per-subwarp kernel: work-group size
constexpr int kRowU = 4;          // rows per subwarp in the row-per-subwarp kernel
constexpr int kRowMaxRows = 32768;  // larger matrices take the load-balanced kernel
constexpr int64_t kStageMinNnz = 8192;  // staged-rows kernel: fewer entries take the load-balanced kernel

// In csr_cb_tiles of a solver's own copy of a matrix (the solvers do not use the
// column-blocked copy): not the staged-rows kernel, but the tile kernel and, up
// to 2 kRowMaxRows rows, the row-per-subwarp kernel. BiCG sets it above
// kRowMaxRows rows and BiCGSTAB above kBicgstabStageRows: their residuals jump
// about, so that sums in another order move the solution at the tolerance, the
// further the longer the solve. Staged or other sums against these, convection-
// diffusion, one entry over the RMS and the norm: BiCG up to 32^3 rows 3e-8 and
// 4e-10, 36^3 to 118^3 up to 9e-8 and 1e-9; BiCGSTAB up to 63^3 1e-10 of the
// norm, 81^3 to 118^3 1.2e-9. CG, GMRES and pipelined CG: 2e-9 and 6e-10 at any
// size.
constexpr int32_t kCsrNoStage = -1;
constexpr int64_t kBicgstabStageRows = 1 << 18;

inline int64_t csr_tiles(int64_t nnz) { return nnz > 0 ? ceil_div(nnz, kCsrTile) : 1; }

struct KState;

// Subwarp width of the row-per-subwarp kernel for A, or 0 when A takes
// another kernel: the staged-rows kernel does not take A, A is small (at most
// kRowMaxRows rows) and its rows are short and even (max_row_len known and at
// most twice the power of two at or above the mean row length).
int csr_rows_sub(const spx_matrix &A);
// Number of dot partials the CSR product with epi > 0 writes for A.
int64_t csr_dot_parts(const spx_matrix &A);
// The most that any of the CSR kernels writes for a matrix of this size: a
// work-group takes 2048 entries (tiles) or, at most 2048 of them, 16 rows or
// more (row-per-subwarp: up to kRowMaxRows rows; staged rows: a grid of up to
// 1024).
inline int64_t csr_dot_parts_most(int64_t nrows, int64_t nnz)
{
    const int64_t rows = pad_to_xcds(ceil_div(nrows, 16)), tiles = csr_tiles(nnz);
    const int64_t most = rows < 2048 ? rows : 2048;
    return most > tiles ? most : tiles;
}

// Writes the tile partition (2 * (csr_tiles(nnz) + 1) int32) of A.
spx_status csr_partition_launch(const spx_matrix &A, int32_t *part, hipStream_t stream);
inline int64_t csr_partition_bytes(int64_t nnz) { return 2 * (csr_tiles(nnz) + 1) * (int64_t)sizeof(int32_t); }

// y = alpha*A*x + beta*y for a CSR matrix with stored value type V and vector
// type X. epi = 1: also sum_i y_i*dot_with_i; epi = 2: that and sum_i y_i^2, in
// epi rows of csr_dot_parts(A) partials (one per work-group, fixed order), which
// the caller sums. With a solver state st, a set st->flag skips the work.
template <typename V, typename X>
spx_status csr_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, const X *dot_with,
                           X *dot_partials, hipStream_t stream, int epi = 0, KState *st = nullptr, int op = 0);

}  // namespace spx
