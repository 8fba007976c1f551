// spmv_formats.hip -- COO, ELL and hybrid ELL+COO products for gfx950.
//
// COO (Section 4: the Coo product "relies on atomic operations"): entries
// sorted by row are cut into wavefront spans of a few chunks of 4 or 8 tiles
// of 64 entries. A wavefront walks its span chunk by chunk (all loads of a chunk
// issued first) in 64-entry tiles: coalesced loads of row, column and value,
// gathered x, then one segmented inclusive scan across the 64 lanes (DPP row
// shifts + row broadcasts, wave.hpp) keyed by the row index. The last segment
// of a tile is carried in registers into the next tile and chunk. A row
// wholly inside a span is written with a plain store; a row that crosses a
// span boundary is accumulated with a float atomic add after a small pre-pass
// has set it to beta*y (the only non-deterministic order).
// Rows without entries (gaps between consecutive row indices) are written
// beta*y by the chunk that sees the gap.
//
// ELL: slot-major layout (slot k of row i at k*ld + i), one lane per row,
// so every slot load is a contiguous 64-lane access. Padding slots (column -1)
// skip the gather; since padding follows a row's entries, a wavefront stops
// as soon as all of its rows have reached padding.
//
// HYB: the ELL kernel writes y = alpha*A_ell*x + beta*y, then the COO kernel
// adds the COO part (plain read-modify-write for rows inside a chunk, atomics
// for rows crossing a chunk boundary).
#include "common.hpp"
#include "krylov.hpp"
#include "spmv.hpp"
#include "wave.hpp"

namespace spx {

constexpr int kEllSlots = 4;   // slot columns a thread has in flight (ELL: of two rows, mostly)
constexpr int kSellSlots = 8;  // the same, SELL-P

template <typename X>
__device__ __forceinline__ X scaled(X v, X beta)
{
    return beta == X(0) ? X(0) : beta * v;
}

// Pre-pass: a row crossing a chunk boundary is set to beta*y exactly once,
// by the first boundary that falls strictly inside it.
template <typename X>
__global__ __launch_bounds__(256) void coo_split_init_kernel(int64_t nnz, int64_t nspans, int64_t span,
                                                            const int32_t *__restrict__ row, X *__restrict__ y,
                                                            X beta)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x + 1;  // boundary k*span, k >= 1
    if (k >= nspans) return;
    const int64_t b = k * span;
    const int32_t r = row[b];
    if (row[b - 1] != r) return;                  // boundary between rows: no split
    if (k >= 2 && row[b - span - 1] == r) return;  // an earlier boundary is inside r too
    y[r] = beta == X(0) ? X(0) : beta * y[r];
}

template <typename X>
__global__ __launch_bounds__(256) void scale_kernel(int64_t n, X *__restrict__ y, X beta)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = scaled(y[i], beta);
}

// The sum of row r, which lies inside one span. kBetaZero: beta == 0, so y is
// written without being read (no dependent load in the tile loop).
template <typename X, bool kAccumulate, bool kBetaZero>
__device__ __forceinline__ void coo_write(int32_t r, X sum, X *__restrict__ y, X alpha, X beta)
{
    if (kAccumulate) {
        y[r] += alpha * sum;
    } else if (kBetaZero) {
        y[r] = alpha * sum;
    } else {
        y[r] = alpha * sum + scaled(y[r], beta);
    }
}

// What bounds it: the gathers on scattered columns, the scan of short segments
// on stencils. The first row's atomic add waits for the span's end: issued
// where the row closes it held up every later load of the span. Random rows of
// 5 to 45 entries, 400,000 rows, float64 88.7 -> 62.2 us (rows that never
// cross a span: 57.4 either way), 7-point 160^3 135 -> 118, 27-point 100^3
// 121 -> 102.
// 8 tiles: three wavefronts per SIMD (the loads in flight are enough, and
// fewer rows' gathers share the L2 caches): Zipf rows, 153 million entries,
// float32 1008 -> 980 us; on stencils with 4 tiles it loses 20 %.
// kTogether: a chunk's gathers go out together; otherwise tile by tile.
template <typename V, typename X, bool kAccumulate, bool kBetaZero, int kCooTiles, bool kTogether>
__global__ __launch_bounds__(kCooThreads)
__attribute__((amdgpu_waves_per_eu(kCooTiles == kCooTilesLarge ? 3 : 1, kCooTiles == kCooTilesLarge ? 3 : 8)))
void coo_spmv_kernel(int32_t nrows, int64_t nnz, int64_t nspans,
                                                               int64_t span, int64_t grid_padded,
                                                               const int32_t *__restrict__ row,
                                                               const int32_t *__restrict__ col,
                                                               const V *__restrict__ val, const X *__restrict__ x,
                                                               X *__restrict__ y, X alpha, X beta)
{
    constexpr int kCooChunk = kCooTiles * kWave;  // entries per wavefront chunk
    const int lane = lane_id();
    const int64_t blk = xcd_remap(blockIdx.x, grid_padded);
    const int64_t w = blk * (kCooThreads / kWave) + threadIdx.x / kWave;
    if (w >= nspans) return;
    // this wavefront's span [s0, s1): consecutive chunks of kCooChunk entries
    // whose open row is carried from chunk to chunk in registers; only rows
    // crossing the span's ends need atomics, and those wait for the span's
    // end: loads wait for every atomic issued before them
    const int64_t s0 = w * span;
    const int64_t s1 = (s0 + span < nnz) ? s0 + span : nnz;
    const int32_t row_before = s0 > 0 ? row[s0 - 1] : -1;
    const int32_t row_after = s1 < nnz ? row[s1] : -1;

    int32_t carry_row = -1;
    X carry_val = X(0);
    bool open_left = false;  // the span's first row began before it and has not closed yet
    bool first_pending = false;
    X first_val = X(0);  // its sum, once closed
    for (int64_t c0 = s0; c0 < s1; c0 += kCooChunk) {
        const int64_t c1 = (c0 + kCooChunk < s1) ? c0 + kCooChunk : s1;
        // issue every load of the chunk first (memory-level parallelism); the
        // chunk base is wave-uniform so the loads use scalar base + 32-bit offsets
        const int32_t *__restrict__ rowc = row + c0;
        const int32_t *__restrict__ colc = col + c0;
        const V *__restrict__ valc = val + c0;
        const int cn = (int)(c1 - c0);
        int32_t r[kCooTiles], c[kCooTiles];
        X p[kCooTiles];
#pragma unroll
        for (int t = 0; t < kCooTiles; ++t) {
            const int o = t * kWave + lane;
            r[t] = -1;
            c[t] = 0;
            p[t] = X(0);
            if (o < cn) {
                r[t] = ld_stream(rowc + o);
                c[t] = ld_stream(colc + o);
                p[t] = widen(ld_stream(valc + o));
            }
        }
        const int32_t chunk_before = c0 > 0 ? row[c0 - 1] : -1;
        if constexpr (kTogether) {
            // a load under a per-lane branch together with its use would be
            // waited for before the next one is issued
            X xv[kCooTiles];
#pragma unroll
            for (int t = 0; t < kCooTiles; ++t) xv[t] = x[c[t]];  // column 0 past the end
#pragma unroll
            for (int t = 0; t < kCooTiles; ++t) p[t] = r[t] >= 0 ? p[t] * xv[t] : X(0);
        } else {
#pragma unroll
            for (int t = 0; t < kCooTiles; ++t)
                if (r[t] >= 0) p[t] *= x[c[t]];
        }

#pragma unroll
        for (int t = 0; t < kCooTiles; ++t) {
            const int64_t tb = c0 + t * kWave;
            if (tb >= c1) break;
            const int64_t e = tb + lane;
            const bool valid = e < c1;
            const int32_t rr = r[t];
            const int32_t r0 = readlane(rr, 0);
            if (c0 == s0 && t == 0) open_left = r0 == row_before;
            // the carried segment ends before this tile: write it
            if (carry_row >= 0 && r0 != carry_row) {
                if (open_left) {
                    first_val = carry_val;
                    first_pending = true;
                    open_left = false;
                } else if (lane == 0) {
                    coo_write<X, kAccumulate, kBetaZero>(carry_row, carry_val, y, alpha, beta);
                }
                carry_row = -1;
            }
            const bool merged = (carry_row >= 0);  // lane 0 continues the carried segment
            const int32_t first_prev = (t == 0) ? chunk_before : readlane(r[t > 0 ? t - 1 : 0], kWave - 1);
            const int32_t rprev = wave_shift_up1(rr, first_prev);
            const bool head = !valid || lane == 0 || rr != rprev;
            X v = p[t];
            if (lane == 0 && merged) v += carry_val;
            // gaps: rows strictly between the previous entry's row and this one are empty
            if (!kAccumulate && valid && rr != rprev)
                for (int32_t g = rprev + 1; g < rr; ++g) y[g] = kBetaZero ? X(0) : scaled(y[g], beta);
            if (!kAccumulate && valid && e == nnz - 1)
                for (int32_t g = rr + 1; g < nrows; ++g) y[g] = kBetaZero ? X(0) : scaled(y[g], beta);
            const X sv = wave_segscan(v, head);
            // the last valid lane of the tile and the segment it closes are carried on
            const int tail_e = (c1 - tb < kWave) ? (int)(c1 - tb - 1) : kWave - 1;
            // a lane closes a segment when the next lane starts a new one
            const int32_t rn = wave_shift_down1(rr, -2);
            bool closes = lane < tail_e && rn != rr;
            if (open_left) {
                const lane_mask_t m = ballot64(closes);
                if (m != 0) {
                    const int src = __builtin_ctzll(m);
                    first_val = readlane(sv, src);
                    first_pending = true;
                    open_left = false;
                    closes = closes && lane != src;
                }
            }
            if (closes) coo_write<X, kAccumulate, kBetaZero>(rr, sv, y, alpha, beta);
            carry_row = readlane(rr, tail_e);
            carry_val = readlane(sv, tail_e);
        }
    }
    if (lane != 0) return;
    if (carry_row >= 0) {
        if (open_left || carry_row == row_after) unsafeAtomicAdd(y + carry_row, alpha * carry_val);
        else coo_write<X, kAccumulate, kBetaZero>(carry_row, carry_val, y, alpha, beta);
    }
    if (first_pending) unsafeAtomicAdd(y + row_before, alpha * first_val);
}

// How the ELL product takes the gathers of x (the rule: ell_mode).
enum EllMode : int {
    kEllTogether = 0,  // those of kEllSlots slot columns in flight together
    kEllByRows = 1,    // apart where a wavefront's rows are scattered, else together
    kEllApart = 2      // one of a wavefront in flight at a time
};

// Slots [k, k + kEllSlots) of rows i .. i + kR - 1: columns (-1: no entry) and values.
template <typename V, int kR>
struct EllSlots {
    typedef int32_t CR __attribute__((ext_vector_type(kR)));
    typedef V VR __attribute__((ext_vector_type(kR)));
    CR c[kEllSlots];
    VR v[kEllSlots];

    __device__ __forceinline__ void load(int32_t nrows, int32_t K, int64_t ld, int64_t i, int32_t k,
                                         const int32_t *__restrict__ ecol, const V *__restrict__ eval)
    {
#pragma unroll
        for (int u = 0; u < kEllSlots; ++u) {
            if (k + u >= K) break;
            const int64_t q = (int64_t)(k + u) * ld + (i < nrows ? i : 0);
            c[u] = ld_stream(reinterpret_cast<const CR *>(ecol + q));
            v[u] = ld_stream(reinterpret_cast<const VR *>(eval + q));
        }
    }
    // Drops what lies outside the matrix; false: every row of the wavefront
    // is into its padding.
    __device__ __forceinline__ bool live(int32_t nrows, int32_t K, int64_t i, int32_t k)
    {
        bool any = false;
#pragma unroll
        for (int u = 0; u < kEllSlots; ++u)
#pragma unroll
            for (int r = 0; r < kR; ++r) {
                if (!(k + u < K && i + r < nrows)) c[u][r] = -1;
                if (u == kEllSlots - 1) any |= c[u][r] >= 0;
            }
        return ballot64(any) != 0;
    }
};

// Whether the wavefront's rows have unrelated columns: fewer than a quarter of
// them have their second entry (column c, -1: none) within 16 columns of that
// of the row before.
__device__ __forceinline__ bool scattered_rows(int32_t c)
{
    const int32_t before = wave_shift_up1(c, -1), d = c - before;
    return __popcll(ballot64(c >= 0 && before >= 0 && d <= 16 && d >= -16)) < kWave / 4;
}

// The row sums, kEllSlots slot columns' gathers in flight together (under the
// branch of its use a gather would be waited for alone). The next slots are
// loaded kAhead = 0: after them, 1: before them, once some row is known to
// have more, 2: before this block's columns are known. s: the first slots,
// loaded.
template <int kAhead, typename V, typename X, int kR>
__device__ __forceinline__ void ell_together(EllSlots<V, kR> &s, int32_t nrows, int32_t K, int64_t ld, int64_t i,
                                             const int32_t *__restrict__ ecol, const V *__restrict__ eval,
                                             const X *__restrict__ x, X (&sum)[kR])
{
    EllSlots<V, kR> next;
    for (int32_t k = 0;; k += kEllSlots) {
        bool more = k + kEllSlots < K;
        if (kAhead == 2 && more) next.load(nrows, K, ld, i, k + kEllSlots, ecol, eval);
        const bool live = s.live(nrows, K, i, k);
        more = more && live;
        if (kAhead == 1 && more) next.load(nrows, K, ld, i, k + kEllSlots, ecol, eval);
        X xv[kEllSlots][kR];
#pragma unroll
        for (int u = 0; u < kEllSlots; ++u)
#pragma unroll
            for (int r = 0; r < kR; ++r) {
                xv[u][r] = X(0);
                if (s.c[u][r] >= 0) xv[u][r] = x[s.c[u][r]];
            }
#pragma unroll
        for (int u = 0; u < kEllSlots; ++u)
#pragma unroll
            for (int r = 0; r < kR; ++r)
                if (s.c[u][r] >= 0) sum[r] += widen(s.v[u][r]) * xv[u][r];
        if (!more) return;
        if (kAhead == 0) s.load(nrows, K, ld, i, k + kEllSlots, ecol, eval);
        else s = next;
    }
}

// The same sums with one gather of a wavefront in flight at a time, the loads
// of four slot columns before them.
template <typename V, typename X, int kR>
__device__ __forceinline__ void ell_apart(int32_t nrows, int32_t K, int64_t ld, int64_t i,
                                          const int32_t *__restrict__ ecol, const V *__restrict__ eval,
                                          const X *__restrict__ x, X (&sum)[kR])
{
    typedef typename EllSlots<V, kR>::CR CR;
    typedef typename EllSlots<V, kR>::VR VR;
    const bool in = i < nrows;
    constexpr int U = kEllSlots;
    for (int k = 0; k < K; k += U) {
        CR c[U];
        VR v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int r = 0; r < kR; ++r) {
                c[u][r] = -1;
                v[u][r] = V(0);
            }
            if (in && k + u < K) {
                const int64_t q = (int64_t)(k + u) * ld + i;
                c[u] = ld_stream(reinterpret_cast<const CR *>(ecol + q));
                v[u] = ld_stream(reinterpret_cast<const VR *>(eval + q));
#pragma unroll
                for (int r = 1; r < kR; ++r)
                    if (i + r >= nrows) c[u][r] = -1;  // a slot past the last row is not the matrix's
            }
        }
        bool live = false;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < kR; ++r)
                if (c[u][r] >= 0) sum[r] += widen(v[u][r]) * x[c[u][r]];
#pragma unroll
        for (int r = 0; r < kR; ++r) live |= c[U - 1][r] >= 0;
        if (ballot64(live) == 0) break;  // every row of the wavefront is into its padding
    }
}

// One thread per kR consecutive rows (kR = 2 loads the two rows' slots as
// one vector when ld is even and the arrays are aligned); a wavefront stops
// once all its rows are into their padding.
// What bounds it: the slot stream on banded matrices, there 4.9 to 5.9 TB/s;
// where the columns are scattered, the gathers. kEllByRows, float32: pairs
// where the rows are scattered, otherwise one row per lane in kR passes (a
// pair's gathers share lines).
// kEpi: 0 = plain product; 1 = also the block's sum of y_i*w_i; 2 = that and
// the sum of y_i^2 (one partial per work-group, reduced later in a fixed
// order; a set solver flag skips the launch).
template <typename V, typename X, int kEpi, int kR, EllMode kMode>
__global__ __launch_bounds__(kEllThreads, kMode == kEllByRows ? 8 : 1) void ell_spmv_kernel(int32_t nrows, int32_t K, int64_t ld,
                                                               int64_t grid_padded, const int32_t *__restrict__ ecol,
                                                               const V *__restrict__ eval, const X *__restrict__ x,
                                                               X *__restrict__ y, X alpha, X beta,
                                                               const X *__restrict__ dot_with,
                                                               X *__restrict__ partials, const KState *st)
{
    if (st != nullptr && st->flag != kRunning) return;
    const int64_t nblocks = ((int64_t)nrows + kEllThreads * kR - 1) / (kEllThreads * kR);
    const int64_t blk = xcd_remap(blockIdx.x, grid_padded);
    if (blk >= nblocks) return;
    const int64_t i0 = (blk * kEllThreads + threadIdx.x) * kR;
    X sum[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) sum[r] = X(0);
    int64_t row[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) row[r] = i0 + r;
    if constexpr (kMode == kEllApart) {
        ell_apart(nrows, K, ld, i0, ecol, eval, x, sum);
    } else if (K > 0) {
        // binary16: the test reads the first slots themselves (a load before
        // them costs a 27-point product 3 %); wider ones hold too many
        // registers across it
        constexpr bool kFirst = kMode == kEllTogether || sizeof(V) == 2;
        EllSlots<V, kR> s;
        bool apart = false;
        if constexpr (kFirst) s.load(nrows, K, ld, i0, 0, ecol, eval);
        if constexpr (kMode == kEllByRows) {
            int32_t c = -1;  // of the second slot
            if constexpr (kFirst) {
                if (K > 1) c = s.c[1][0];
            } else {
                if (K > 1 && i0 < nrows) c = ecol[ld + i0];
            }
            apart = scattered_rows(c);
        }
        if (apart) {
            ell_apart(nrows, K, ld, i0, ecol, eval, x, sum);
        } else if constexpr (kMode == kEllByRows && kR > 1 && sizeof(V) == sizeof(float)) {
            const int64_t wave0 = (blk * kEllThreads + (threadIdx.x & ~(kWave - 1))) * kR;
#pragma unroll
            for (int r = 0; r < kR; ++r) {
                EllSlots<V, 1> t;
                X one[1] = {X(0)};
                row[r] = wave0 + r * kWave + lane_id();
                t.load(nrows, K, ld, row[r], 0, ecol, eval);
                ell_together<0>(t, nrows, K, ld, row[r], ecol, eval, x, one);
                sum[r] = one[0];
            }
        } else {
            if constexpr (!kFirst) s.load(nrows, K, ld, i0, 0, ecol, eval);
            ell_together<kMode == kEllTogether ? 2 : (kFirst ? 1 : 0)>(s, nrows, K, ld, i0, ecol, eval, x, sum);
        }
    }
    X d1 = X(0), d2 = X(0);
#pragma unroll
    for (int r = 0; r < kR; ++r) {
        const int64_t i = row[r];
        if (i < nrows) {
            X out = alpha * sum[r];
            if (beta != X(0)) out += beta * y[i];  // y is not read when beta == 0
            y[i] = out;
            if constexpr (kEpi >= 1) d1 += out * dot_with[i];
            if constexpr (kEpi >= 2) d2 += out * out;
        }
    }
    if constexpr (kEpi > 0) {
        __shared__ X s_red[kEllThreads / kWave];
        X v[kEpi];
        v[0] = block_sum<X, kEllThreads>(d1, s_red);
        if constexpr (kEpi >= 2) v[kEpi - 1] = block_sum<X, kEllThreads>(d2, s_red);
        write_partials<X, kEpi>(v, partials, nblocks, blk);
    }
}

template <typename V, typename X, bool kAccumulate>
static spx_status coo_part(int32_t nrows, int32_t ncols, int64_t nnz, const int32_t *row, const int32_t *col, const V *val,
                           const X *x, X *y, X alpha, X beta, hipStream_t stream)
{
    if (nnz == 0) {
        if (!kAccumulate) {
            scale_kernel<X><<<(unsigned)ceil_div(nrows, 256), 256, 0, stream>>>(nrows, y, beta);
            SPX_LAUNCHED();
        }
        return SPX_OK;
    }
    // chunks per wavefront span: enough spans to fill the GPU several times
    // over, at most `most` chunks (fewer spans, fewer boundary atomics)
    const bool large = nnz >= kCooLargeNnz && ncols * (int64_t)sizeof(X) <= kCooCachedX;
    const bool missing = nnz >= kCooLargeNnz && !large;
    const int64_t chunk = (int64_t)kWave * (large ? kCooTilesLarge : kCooTilesSmall);
    const int64_t most = large ? kCooSpanLarge : kCooSpanSmall;
    const int64_t nchunks = ceil_div(nnz, chunk);
    int64_t per = ceil_div(nchunks, kCooTargetSpans);
    per = per < 1 ? 1 : (per > most ? most : per);
    const int64_t span = per * chunk;
    const int64_t nspans = ceil_div(nnz, span);
    if (!kAccumulate && nspans > 1) {
        coo_split_init_kernel<X><<<(unsigned)ceil_div(nspans - 1, 256), 256, 0, stream>>>(nnz, nspans, span, row, y,
                                                                                          beta);
        SPX_LAUNCHED();
    }
    const int64_t blocks = ceil_div(nspans, kCooThreads / kWave);
    const int64_t grid = pad_to_xcds(blocks);
#define SPX_COO_LAUNCH(BZ, TILES, TOGETHER)                                                                         \
    coo_spmv_kernel<V, X, kAccumulate, BZ, TILES, TOGETHER><<<(unsigned)grid, kCooThreads, 0, stream>>>(            \
        nrows, nnz, nspans, span, grid, row, col, val, x, y, alpha, beta)
    if (!kAccumulate && beta == X(0)) {
        if (large) SPX_COO_LAUNCH(!kAccumulate, kCooTilesLarge, true);
        else if (missing) SPX_COO_LAUNCH(!kAccumulate, kCooTilesSmall, false);
        else SPX_COO_LAUNCH(!kAccumulate, kCooTilesSmall, true);
    } else {
        if (large) SPX_COO_LAUNCH(false, kCooTilesLarge, true);
        else if (missing) SPX_COO_LAUNCH(false, kCooTilesSmall, false);
        else SPX_COO_LAUNCH(false, kCooTilesSmall, true);
    }
#undef SPX_COO_LAUNCH
    SPX_LAUNCHED();
    return SPX_OK;
}

template <typename V, typename X>
spx_status coo_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream)
{
    return coo_part<V, X, false>(A.nrows, A.ncols, A.nnz, A.rowidx, A.colidx, static_cast<const V *>(A.vals), x, y, alpha,
                                 beta, stream);
}

// Up to kEllLargeRows rows (two work-groups of pairs per CU) the gathers of a
// few wavefronts have to go out together. Above, where the columns are
// scattered, one in flight per wavefront is better: all wavefronts walk the
// rows' sorted entries side by side, and the window of x they share stays
// small (900,000 rows of 16 random columns: 3.0 million L2 misses, 5.4 with
// four slot columns together). Rows of 5 to 45 random entries, float64, apart
// / together: 250,000 rows 43.6 / 39.2 us, 400,000 rows 55.3 / 71.5, 900,000
// rows 141 / 155; 16 per row, 400,000 rows 39.7 / 47.6. Banded rows want them
// together at any size (7-point 160^3 float64 74 / 70, float32 52 / 45,
// binary16 45 / 40). Ragged rows (a quarter to half of the slots stored) are
// taken as scattered; where padding is most of the stream the loads ahead
// matter more (300,000 Zipf rows, float64 12.4 ms apart, 5.3 together);
// otherwise every wavefront looks at its own rows, but
// for binary16 rows of fewer than 8 entries, too short to pay for it.
constexpr int32_t kEllLargeRows = 1 << 18;
static EllMode ell_mode(const spx_matrix &A)
{
    if (A.nrows <= kEllLargeRows) return kEllTogether;
    const int64_t stored = A.fmt == SPX_HYB ? A.nnz - A.coo_nnz : A.nnz;
    const int64_t slots = (int64_t)A.ell_width * A.nrows;
    if (4 * stored < slots) return kEllTogether;
    if (2 * stored < slots) return kEllApart;
    return A.val_type == SPX_F16 && A.ell_width < 8 ? kEllTogether : kEllByRows;
}

// Two rows per thread when the slot columns can be read two rows at a time:
// even leading dimension (so a pair never straddles a slot column; with an
// odd nrows the last pair's second row is in-bounds padding) and arrays
// aligned to two entries. Float32 gathered together takes one row per lane: a
// pair's gathers share lines, and the stream is better off without.
// Pairs against single rows, cold: 27-point 100^3 float64 61.5 / 62.6 us,
// float32 50.2 / 38.1, binary16 36.4 / 41.6; 7-point 160^3 float64 70.8 / 70.7,
// float32 50.2 / 44.6, binary16 40.2 / 49.2.
static int ell_rows_per_thread(const spx_matrix &A)
{
    const size_t sv = A.val_type == SPX_F64 ? 8 : (A.val_type == SPX_F32 ? 4 : 2);
    const bool even = (A.ell_ld % 2) == 0;
    const bool aligned = (reinterpret_cast<uintptr_t>(A.ell_col) % 8 == 0) &&
                         (reinterpret_cast<uintptr_t>(A.ell_val) % (2 * sv) == 0);
    return even && aligned && (A.val_type != SPX_F32 || ell_mode(A) != kEllTogether) ? 2 : 1;
}

int64_t ell_dot_parts(const spx_matrix &A)
{
    return A.nrows > 0 ? ceil_div(A.nrows, (int64_t)kEllThreads * ell_rows_per_thread(A)) : 1;
}

template <typename V, typename X>
spx_status ell_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream, int epi,
                           const X *dot_with, X *partials, const KState *st)
{
    const int kr = ell_rows_per_thread(A);
    const int64_t blocks = ceil_div(A.nrows, (int64_t)kEllThreads * kr);
    const int64_t grid = pad_to_xcds(blocks);
#define SPX_ELL_LAUNCH(E, R)                                                                                        \
    switch (ell_mode(A)) {                                                                                          \
    case kEllTogether: SPX_ELL_KERNEL(E, R, kEllTogether); break;                                                   \
    case kEllByRows: SPX_ELL_KERNEL(E, R, kEllByRows); break;                                                       \
    default: SPX_ELL_KERNEL(E, R, kEllApart); break;                                                                \
    }
#define SPX_ELL_KERNEL(E, R, L)                                                                                     \
    ell_spmv_kernel<V, X, E, R, L><<<(unsigned)grid, kEllThreads, 0, stream>>>(                                        \
        A.nrows, A.ell_width, A.ell_ld, grid, A.ell_col, static_cast<const V *>(A.ell_val), x, y, alpha, beta,      \
        dot_with, partials, st)
    if (kr == 2) {
        if (epi == 2) { SPX_ELL_LAUNCH(2, 2) }
        else if (epi == 1) { SPX_ELL_LAUNCH(1, 2) }
        else { SPX_ELL_LAUNCH(0, 2) }
    } else {
        if (epi == 2) { SPX_ELL_LAUNCH(2, 1) }
        else if (epi == 1) { SPX_ELL_LAUNCH(1, 1) }
        else { SPX_ELL_LAUNCH(0, 1) }
    }
#undef SPX_ELL_KERNEL
#undef SPX_ELL_LAUNCH
    SPX_LAUNCHED();
    return SPX_OK;
}

template <typename V, typename X>
spx_status hyb_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream)
{
    SPX_CHECK(ell_spmv_launch<V, X>(A, x, y, alpha, beta, stream));
    return coo_part<V, X, true>(A.nrows, A.ncols, A.coo_nnz, A.rowidx, A.colidx, static_cast<const V *>(A.vals), x, y, alpha,
                                beta, stream);
}

// What bounds the SELL-P products: the slot stream (see the ELL kernel).
// Before -> after, 64-row slices: 27-point 101^3 float32 48.9 -> 39.1 us
// (5.9 TB/s), float64 67.6 -> 64.6, 7-point 160^3 binary16 60.5 -> 39.3 us.
// 4, 6 and 12 slot columns at a time, the same cases: 37.7 / 37.5 / 41.9,
// 62.3 / 62.6 / 65.8 and 46.4 / 50.3 / 46.8 us against 38.1, 64.0 and 39.6.
// One row's sum over slot columns k, k + step, ... below w (slot column k of
// the row at k * C): kSellSlots columns at a time, the next ones loaded while
// this block's gathers are in flight. Columns past the last are read again
// and dropped; the entries are added in order.
// kByRows (64-row slices, step 1): a wavefront of scattered rows takes one
// gather at a time instead.
template <bool kByRows, typename V, typename X>
__device__ __forceinline__ X slot_sum(const int32_t *__restrict__ cs, const V *__restrict__ vs, int32_t k,
                                      int32_t step, int32_t w, int32_t C, const X *__restrict__ x)
{
    constexpr int U = kSellSlots;
    X sum = X(0);
    if (k >= w) return sum;
    auto load = [&](int32_t j, int32_t(&c)[U], V(&v)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = (int64_t)(j + u * step < w ? j + u * step : j) * C;
            c[u] = ld_stream(cs + q);
            v[u] = ld_stream(vs + q);
        }
    };
    int32_t cc[U], cn[U];
    V vv[U], vn[U];
    load(k, cc, vv);
    if (kByRows && scattered_rows(cc[1])) {
        while (true) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u * step < w && cc[u] >= 0) sum += widen(vv[u]) * x[cc[u]];
            k += U * step;
            if (k >= w) return sum;
            load(k, cc, vv);
        }
    }
    while (true) {
        const int32_t next = k + U * step;
        if (next < w) load(next, cn, vn);
        X xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k + u * step >= w) cc[u] = -1;
            xv[u] = X(0);
            if (cc[u] >= 0) xv[u] = x[cc[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (cc[u] >= 0) sum += widen(vv[u]) * xv[u];
        if (next >= w) return sum;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cc[u] = cn[u];
            vv[u] = vn[u];
        }
        k = next;
    }
}

// SELL-P: one work-group of kSellThreads per slice. Lane l = tid % C owns row
// s*C + l; the G = kSellThreads / C lane groups take the slice's slot
// columns round robin (group g: columns g, g + G, ...), each slot column
// read coalesced across the lanes; the G partial sums of a row are added in
// group order. Padding slots (column -1) contribute nothing.
// kEpi: 0 = plain product; 1 = also the slice's sum of y_i*w_i; 2 = that and
// sum of y_i^2 (one partial per slice, reduced later in a fixed order; a set
// solver flag skips the launch).
template <typename V, typename X, int kEpi>
__global__ __launch_bounds__(kSellThreads) void sellp_spmv_kernel(int32_t nrows, int32_t C, int32_t log2c,
                                                                 int64_t nslices, int64_t grid_padded,
                                                                 const int32_t *__restrict__ sets,
                                                                 const int32_t *__restrict__ scol,
                                                                 const V *__restrict__ sval, const X *__restrict__ x,
                                                                 X *__restrict__ y, X alpha, X beta,
                                                                 const X *__restrict__ dot_with,
                                                                 X *__restrict__ partials, const KState *st)
{
    if (st != nullptr && st->flag != kRunning) return;
    __shared__ X part[kSellThreads];
    const int64_t s = xcd_remap(blockIdx.x, grid_padded);
    if (s >= nslices) return;
    const int tid = threadIdx.x;
    const int l = tid & (C - 1), g = tid >> log2c;
    const int G = kSellThreads >> log2c;
    const int32_t k0 = sets[s], w = sets[s + 1] - k0;
    const int32_t *__restrict__ cs = scol + (int64_t)k0 * C + l;
    const V *__restrict__ vs = sval + (int64_t)k0 * C + l;
    const X sum = slot_sum<false>(cs, vs, g, G, w, C, x);
    part[tid] = sum;
    __syncthreads();
    const int64_t row = s * C + l;
    X d1 = X(0), d2 = X(0);
    if (g == 0 && row < nrows) {
        X t = part[l];
        for (int j = 1; j < G; ++j) t += part[j * C + l];
        X out = alpha * t;
        if (beta != X(0)) out += beta * y[row];
        y[row] = out;
        if constexpr (kEpi >= 1) d1 = out * dot_with[row];
        if constexpr (kEpi >= 2) d2 = out * out;
    }
    if constexpr (kEpi > 0) {
        __shared__ X s_red[kSellThreads / kWave];
        X v[kEpi];
        v[0] = block_sum<X, kSellThreads>(d1, s_red);
        if constexpr (kEpi >= 2) v[kEpi - 1] = block_sum<X, kSellThreads>(d2, s_red);
        write_partials<X, kEpi>(v, partials, nslices, s);
    }
}

// SELL-P with 64-row slices: one wavefront per slice, one lane per row, eight
// slot columns in flight per lane (the slot columns are read coalesced and,
// on banded matrices, so are the gathers of x); no cross-lane reduction.
template <typename V, typename X, int kEpi, bool kByRows>
__global__ __launch_bounds__(kSellThreads) void sellp64_spmv_kernel(int32_t nrows, int64_t nslices,
                                                                   int64_t grid_padded,
                                                                   const int32_t *__restrict__ sets,
                                                                   const int32_t *__restrict__ scol,
                                                                   const V *__restrict__ sval,
                                                                   const X *__restrict__ x, X *__restrict__ y,
                                                                   X alpha, X beta, const X *__restrict__ dot_with,
                                                                   X *__restrict__ partials, const KState *st)
{
    if (st != nullptr && st->flag != kRunning) return;
    constexpr int kSlices = kSellThreads / kWave;  // slices per work-group
    const int64_t blk = xcd_remap(blockIdx.x, grid_padded);
    const int64_t nblocks = (nslices + kSlices - 1) / kSlices;
    if (blk >= nblocks) return;
    const int64_t s = blk * kSlices + threadIdx.x / kWave;
    const int l = lane_id();
    X d1 = X(0), d2 = X(0);
    if (s < nslices) {
        const int32_t k0 = sets[s], w = sets[s + 1] - k0;
        const int32_t *__restrict__ cs = scol + (int64_t)k0 * kWave + l;
        const V *__restrict__ vs = sval + (int64_t)k0 * kWave + l;
        const X sum = slot_sum<kByRows>(cs, vs, 0, 1, w, kWave, x);
        const int64_t row = s * kWave + l;
        if (row < nrows) {
            X out = alpha * sum;
            if (beta != X(0)) out += beta * y[row];
            y[row] = out;
            if constexpr (kEpi >= 1) d1 = out * dot_with[row];
            if constexpr (kEpi >= 2) d2 = out * out;
        }
    }
    if constexpr (kEpi > 0) {
        __shared__ X s_red[kSellThreads / kWave];
        X v[kEpi];
        v[0] = block_sum<X, kSellThreads>(d1, s_red);
        if constexpr (kEpi >= 2) v[kEpi - 1] = block_sum<X, kSellThreads>(d2, s_red);
        write_partials<X, kEpi>(v, partials, nblocks, blk);
    }
}

// Whether the 64-row slices' wavefronts look for scattered rows (see ell_mode
// for why these are better off with one gather at a time). It pays where the
// rows fill one to two wavefronts per SIMD (rows of 32 random columns,
// 100,000 rows: float64 19.5 us against 24.4 together, float32 13.9 against
// 19.0; 50,000 rows 9.9 together; 24 per row, 200,000 rows, float32 33.7 and
// 31.1), and in float64 where x is larger than one
// XCD's L2 (rows of 5 to 45 random entries, 900,000 rows: 146.6 against 153;
// 400,000 rows 64.2 against 63.2). Slices of fewer than 8 slot columns are too
// short to pay for the look (5-point 1500^2: 37.7 us against 33.9), and where
// padding is most of the stream the loads ahead matter more than the gathers
// (Zipf rows, 3 % of the slots stored: 18.4 ms against 12.8).
static bool sell_by_rows(const spx_matrix &A)
{
    const int64_t slots = A.slice_cols * kWave;
    if (slots < int64_t(8) * A.nrows || 4 * A.nnz < slots) return false;
    return (A.nrows > (1 << 16) && A.nrows <= (1 << 17)) ||
           (A.val_type == SPX_F64 && A.ncols * (int64_t)sizeof(double) > kCooCachedX);
}

int64_t sellp_dot_parts(const spx_matrix &A)
{
    const int64_t ns = A.nrows > 0 ? ceil_div(A.nrows, A.slice_size) : 1;
    return A.slice_size == kWave ? ceil_div(ns, kSellThreads / kWave) : ns;
}

template <typename V, typename X>
spx_status sellp_spmv_launch(const spx_matrix &A, const X *x, X *y, X alpha, X beta, hipStream_t stream, int epi,
                             const X *dot_with, X *partials, const KState *st)
{
    const int32_t C = A.slice_size;
    const int64_t ns = ceil_div(A.nrows, C);
    if (C == kWave) {
        const int64_t nblocks = sellp_dot_parts(A);
        const int64_t grid = pad_to_xcds(nblocks);
#define SPX_SELL64_LAUNCH(E, B)                                                                                    \
    sellp64_spmv_kernel<V, X, E, B><<<(unsigned)grid, kSellThreads, 0, stream>>>(                                  \
        A.nrows, ns, grid, A.slice_sets, A.ell_col, static_cast<const V *>(A.ell_val), x, y, alpha, beta, dot_with, \
        partials, st)
        if (sell_by_rows(A)) {
            if (epi == 2) SPX_SELL64_LAUNCH(2, true);
            else if (epi == 1) SPX_SELL64_LAUNCH(1, true);
            else SPX_SELL64_LAUNCH(0, true);
        } else {
            if (epi == 2) SPX_SELL64_LAUNCH(2, false);
            else if (epi == 1) SPX_SELL64_LAUNCH(1, false);
            else SPX_SELL64_LAUNCH(0, false);
        }
#undef SPX_SELL64_LAUNCH
        SPX_LAUNCHED();
        return SPX_OK;
    }
    int32_t log2c = 0;
    while ((1 << log2c) < C) ++log2c;
    const int64_t grid = pad_to_xcds(ns);
#define SPX_SELL_LAUNCH(E)                                                                                         \
    sellp_spmv_kernel<V, X, E><<<(unsigned)grid, kSellThreads, 0, stream>>>(                                       \
        A.nrows, C, log2c, ns, grid, A.slice_sets, A.ell_col, static_cast<const V *>(A.ell_val), x, y, alpha, beta, \
        dot_with, partials, st)
    if (epi == 2) SPX_SELL_LAUNCH(2);
    else if (epi == 1) SPX_SELL_LAUNCH(1);
    else SPX_SELL_LAUNCH(0);
#undef SPX_SELL_LAUNCH
    SPX_LAUNCHED();
    return SPX_OK;
}

#define SPX_INST(V, X)                                                                                          \
    template spx_status coo_spmv_launch<V, X>(const spx_matrix &, const X *, X *, X, X, hipStream_t);          \
    template spx_status ell_spmv_launch<V, X>(const spx_matrix &, const X *, X *, X, X, hipStream_t, int,        \
                                              const X *, X *, const KState *);                                    \
    template spx_status hyb_spmv_launch<V, X>(const spx_matrix &, const X *, X *, X, X, hipStream_t);          \
    template spx_status sellp_spmv_launch<V, X>(const spx_matrix &, const X *, X *, X, X, hipStream_t, int,      \
                                                const X *, X *, const KState *);
SPX_INST(double, double)
SPX_INST(float, float)
SPX_INST(_Float16, float)
#undef SPX_INST

}  // namespace spx
