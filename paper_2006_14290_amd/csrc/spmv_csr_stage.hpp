// spmv_csr_stage.hpp -- CSR product for rows of similar, known length: every
// wavefront streams its own rows through LDS, with no work-group barrier.
//
// A wavefront takes blocks of kRows * 64 / kSize consecutive rows. The
// block's columns and values lie in one contiguous stretch of the CSR arrays;
// it is copied straight from memory into the wavefront's own LDS slice
// (global_load_lds, 16 bytes per lane, non-temporal: no registers hold the
// stream), then kSize lanes per row read their entries back in row order, so
// that one gather instruction touches x at neighbouring columns, and all
// kRows * kLen gathers of a lane are in flight together. Row pointers of the
// block after next are loaded a block ahead. Entries that a row has beyond
// kSize * kLen, and those past the stage or the last whole 16-byte vector of
// the arrays, are read directly: any row length gives the right sum, only
// long ones give it slowly. Every row is summed by its own lanes in a fixed
// order, and the blocks of a wavefront are fixed by the grid: results are
// bitwise reproducible.
//
// What bounds it: the matrix stream. Against the tile kernel
// (spmv_csr_tile.hpp), which needs four barriers and a register round trip
// per 2048 entries, it keeps the stream going while other wavefronts gather.
// Measured on one MI355X, matrices cold in the Infinity Cache, tile kernel ->
// this one: 27-point 100^3 float64 67.1 -> 63.3 us (5.33 TB/s), float32 45.7
// -> 39.4; 7-point 160^3 float64 85.9 -> 75.0 us (5.65 TB/s), float32 59.5 ->
// 47.6, binary16 values 67.5 -> 42.4.
#pragma once

#include "common.hpp"
#include "krylov.hpp"
#include "spmv_csr.hpp"
#include "wave.hpp"

namespace spx {

constexpr int kStageWaves = 4;  // wavefronts per work-group (each on its own rows)

// Sums that a lane's entries are spread over (1 or 4), so that a row's rounding
// errors grow as in a subwarp's tree and not along one chain of 7 to 16
// entries. RMS error over the RMS of the result, float32, subwarps / one chain
// / four: 7-point 128^3 5.03e-8 / 5.08e-8 / 4.67e-8, 27-point 30^3 6.47e-8 /
// 7.25e-8 / 6.04e-8; the time is the same. float64 rows of one lane keep one
// chain, the order of a plain loop over the row.
template <typename X, int kSize>
constexpr int stage_chains()
{
    return sizeof(X) == 8 && kSize == 1 ? 1 : 4;
}

// 16 bytes per lane from g (per lane) to lds (uniform) + 16 * lane. The
// compiler does not wait for these copies before reading LDS: every use is
// preceded by an explicit s_waitcnt vmcnt(0).
__device__ __forceinline__ void lds_copy16(const void *g, void *lds)
{
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) const void *)g,
                                     (__attribute__((address_space(3))) void *)lds, 16, 0, 2 /* nt */);
}

// nblk: row blocks; kCap: entries a wavefront stages per block (a multiple of
// 512). nnz8: nnz rounded down to whole vectors (> 0). col and val are
// 16-byte aligned. kEpi as in csr_tile, one partial per work-group.
template <typename V, typename X, int kEpi, int kSize, int kRows, int kLen, int kCap>
__global__ __launch_bounds__(kStageWaves *kWave) void csr_stage_kernel(
    int32_t nrows, int32_t nnz8, int32_t nblk, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
    const V *__restrict__ val, const X *__restrict__ x, X *y, X alpha, X beta, const X *__restrict__ dot_with,
    X *__restrict__ dot_partials, const KState *__restrict__ st)
{
    if (st != nullptr && st->flag != kRunning) return;
    constexpr int kGroups = kWave / kSize;        // rows side by side in the wavefront
    constexpr int kBlk = kRows * kGroups;         // rows per block
    constexpr int kVE = 16 / (int)sizeof(V);      // values per vector
    constexpr int kAlign = kVE > 4 ? kVE : 4;     // entries: value and column vectors both start here
    static_assert(kCap % (kWave * kVE) == 0 && kCap % (kWave * 4) == 0, "whole copies only");
    __shared__ __align__(16) unsigned char s_stage[kStageWaves * kCap * (sizeof(V) + sizeof(int32_t))];
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    V *s_val = reinterpret_cast<V *>(s_stage + (size_t)wid * kCap * (sizeof(V) + sizeof(int32_t)));
    int32_t *s_col = reinterpret_cast<int32_t *>(s_val + kCap);
    const int g = lane / kSize, sl = lane % kSize;

    // each XCD takes a contiguous range of blocks, its wavefronts in turn
    const int step = (int)(gridDim.x / kXcds) * kStageWaves;
    const int per = (nblk + kXcds - 1) / kXcds;
    const int b0 = (int)(blockIdx.x % kXcds) * per;
    const int b1 = b0 + per < nblk ? b0 + per : nblk;
    int blk = b0 + (int)(blockIdx.x / kXcds) * kStageWaves + wid;

    auto load_bounds = [&](int b, int32_t(&a)[kRows], int32_t(&e)[kRows]) {
#pragma unroll
        for (int t = 0; t < kRows; ++t) {
            const int64_t r = (int64_t)b * kBlk + t * kGroups + g;
            a[t] = rowptr[r < nrows ? r : nrows];
            e[t] = rowptr[r + 1 < nrows ? r + 1 : nrows];
        }
    };
    // copies entries [s & ~(kAlign-1), + kCap) as far as they lie below e and
    // nnz8; lanes past that repeat the last vector wanted
    auto stage = [&](int32_t s, int32_t e) {
        const int32_t a0 = s & ~(kAlign - 1);
        const int32_t lim = e < nnz8 ? e : nnz8;
        const int32_t last = lim > 0 ? lim - 1 : 0;
        const int32_t lastc = last & ~3, lastv = last & ~(kVE - 1);
#pragma unroll
        for (int u = 0; u < kCap / (4 * kWave); ++u) {
            const int32_t p = a0 + (u * kWave + lane) * 4;
            lds_copy16(col + (p < lastc ? p : lastc), s_col + u * kWave * 4);
        }
#pragma unroll
        for (int u = 0; u < kCap / (kVE * kWave); ++u) {
            const int32_t p = a0 + (u * kWave + lane) * kVE;
            lds_copy16(val + (p < lastv ? p : lastv), s_val + u * kWave * kVE);
        }
    };

    X d1 = X(0), d2 = X(0);
    if (blk < b1) {
        int32_t ra[kRows], rb[kRows], na[kRows], nb[kRows];
        load_bounds(blk, ra, rb);
        int32_t s = __builtin_amdgcn_readfirstlane(ra[0]);
        stage(s, readlane(rb[kRows - 1], kWave - 1));
        int nx = blk + step;
        load_bounds(nx < b1 ? nx : blk, na, nb);
        while (true) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies have landed
            const int32_t a0 = s & ~(kAlign - 1);
            const int32_t lim = nnz8 - a0 > kCap ? a0 + kCap : nnz8;  // staged: [a0, lim)
            int32_t c[kRows][kLen];
            V v[kRows][kLen];
            X xv[kRows][kLen], yv[kRows], wv[kRows];
#pragma unroll
            for (int t = 0; t < kRows; ++t) {
                const int32_t pe = rb[t] < lim ? rb[t] : lim;
#pragma unroll
                for (int u = 0; u < kLen; ++u) {
                    const int32_t p = ra[t] + sl + u * kSize;
                    const int32_t q = p < pe ? p - a0 : 0;
                    c[t][u] = s_col[q];
                    v[t][u] = s_val[q];
                    if (p >= pe) c[t][u] = 0;
                }
            }
#pragma unroll
            for (int t = 0; t < kRows; ++t)
#pragma unroll
                for (int u = 0; u < kLen; ++u) xv[t][u] = x[c[t][u]];
            const int64_t row0 = (int64_t)blk * kBlk + g;
#pragma unroll
            for (int t = 0; t < kRows; ++t) {
                const int64_t row = row0 + t * kGroups;
                yv[t] = wv[t] = X(0);
                if (sl == 0 && row < nrows) {
                    if (beta != X(0)) yv[t] = y[row];  // y is not read when beta == 0
                    if constexpr (kEpi >= 1) wv[t] = dot_with[row];
                }
            }
#pragma unroll
            for (int t = 0; t < kRows; ++t) {
                const int32_t pe = rb[t] < lim ? rb[t] : lim;
                constexpr int kChains = stage_chains<X, kSize>();
                X chain[kChains];
#pragma unroll
                for (int u = 0; u < kChains; ++u) chain[u] = X(0);
#pragma unroll
                for (int u = 0; u < kLen; ++u) {
                    // lanes past the row's end keep their sum (never 0 * inf)
                    const X f = chain[u % kChains] + widen(v[t][u]) * xv[t][u];
                    chain[u % kChains] = ra[t] + sl + u * kSize < pe ? f : chain[u % kChains];
                }
                X sum = chain[0];
                if constexpr (kChains == 4) sum = (chain[0] + chain[1]) + (chain[2] + chain[3]);
                // the row's entries that were not staged or not unrolled
                for (int32_t p = ra[t] + sl + (rb[t] > lim ? 0 : kLen * kSize); p < rb[t]; p += kSize)
                    if (p >= lim || p >= ra[t] + kLen * kSize) sum += widen(val[p]) * x[col[p]];
                sum = subwave_sum<kSize>(sum);
                const int64_t row = row0 + t * kGroups;
                if (sl == 0 && row < nrows) {
                    X out = alpha * sum;
                    if (beta != X(0)) out += beta * yv[t];
                    y[row] = out;
                    if constexpr (kEpi >= 1) d1 += out * wv[t];
                    if constexpr (kEpi >= 2) d2 += out * out;
                }
            }
            if (nx >= b1) break;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this block's LDS reads are done
            s = __builtin_amdgcn_readfirstlane(na[0]);
            stage(s, readlane(nb[kRows - 1], kWave - 1));
#pragma unroll
            for (int t = 0; t < kRows; ++t) {
                ra[t] = na[t];
                rb[t] = nb[t];
            }
            blk = nx;
            nx += step;
            load_bounds(nx < b1 ? nx : blk, na, nb);
        }
    }
    if constexpr (kEpi > 0) {
        __shared__ X s_red[kStageWaves];
        X out[kEpi];
        out[0] = block_sum<X, kStageWaves * kWave>(d1, s_red);
        if constexpr (kEpi >= 2) out[kEpi - 1] = block_sum<X, kStageWaves * kWave>(d2, s_red);
        write_partials<X, kEpi>(out, dot_partials, gridDim.x, blockIdx.x);
    }
}

}  // namespace spx
