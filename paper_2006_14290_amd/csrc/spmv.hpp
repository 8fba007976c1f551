// spmv.hpp -- launch interfaces of the COO, ELL and hybrid products and the
// shared descriptor check.
#pragma once

#include "common.hpp"

namespace spx {

spx_status check_matrix(const spx_matrix *A, const char *who);
// Canonical-form checks of host CSR arrays (spx_validate_csr_host).
spx_status validate_csr_host(int32_t nrows, int32_t ncols, int64_t nnz, const int32_t *rowptr, const int32_t *col);
// colblock: use A's column-blocked copy when it has one (the public product
// entry points); the solvers call it with false (plain CSR product).
spx_status spmv_dispatch(const spx_matrix &A, const void *x, void *y, double alpha, double beta,
                         hipStream_t stream, bool colblock = false);

constexpr int kCooThreads = 256;
// 64-entry tiles per wavefront chunk. Large matrices (kCooLargeNnz entries)
// whose x fits one XCD's L2 (kCooCachedX bytes) take larger chunks and longer
// spans: fewer open rows and atomics, still tens of thousands of spans. Zipf
// rows, float32, 153 million entries: 1028 us with 4 tiles and spans of 8
// chunks, 963 with 8 and 16; 800,000 entries 7.3 / 9.6. With a larger x the
// gathers' line fills bind: more of them in flight take as long or longer
// (float64, 1595 us tile by tile, 1617 with 8 tiles together, cold).
constexpr int kCooTilesSmall = 4, kCooTilesLarge = 8;
constexpr int64_t kCooSpanSmall = 8, kCooSpanLarge = 16;  // chunks per span at most
constexpr int64_t kCooLargeNnz = int64_t(1) << 25;
constexpr int64_t kCooCachedX = int64_t(4) << 20;
constexpr int64_t kCooTargetSpans = 16384;  // wavefront spans to aim for
constexpr int kEllThreads = 256;
constexpr int kSellThreads = 256;

template <typename V, typename X>
spx_status coo_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream);
struct KState;
// epi = 1: also one partial of sum_i y_i*dot_with_i per work-group
// (ell_dot_parts(A) of them); epi = 2: that and sum_i y_i^2; a set st->flag
// skips the launch.
template <typename V, typename X>
spx_status ell_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream, int epi = 0,
                           const X *dot_with = nullptr, X *partials = nullptr, const KState *st = nullptr);
int64_t ell_dot_parts(const spx_matrix &A);
template <typename V, typename X>
spx_status hyb_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream);
// epi = 1: also the partials of sum_i y_i*dot_with_i (sellp_dot_parts(A) of
// them); epi = 2: that and sum_i y_i^2 (partials[epi][parts]); a set
// st->flag skips the launch.
int64_t sellp_dot_parts(const spx_matrix &A);
template <typename V, typename X>
spx_status sellp_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream,
                             int epi = 0, const X *dot_with = nullptr, X *partials = nullptr,
                             const KState *st = nullptr);

}  // namespace spx
