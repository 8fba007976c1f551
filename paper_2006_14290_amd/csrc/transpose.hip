// transpose.hip -- CSR transpose on the device.
//
// In CSR, A^T is A's entries ordered by (column, row). A's entries are
// already in row order, so a stable sort of their column indices yields that
// order. Up to 2^22 columns and 30
// million entries, two steps, most significant digit first:
//   1. a stable partition of the entries (column, row, value) into at most
//      2,048 buckets of consecutive columns: per tile of 4,096 entries a
//      histogram of buckets, prefix sums over the tiles (coalesced: a thread
//      per bucket), then every wavefront ranks its 1,024 entries among equal
//      buckets (ballots on the bucket's bits and its own counters in LDS, no
//      barrier) and writes them out, with the row found by marking the tile's
//      row starts;
//   2. a stable counting sort of every bucket by column: counts per column
//      and wavefront in LDS, a scan (which also gives A^T's row pointer), and
//      the same ranking; the output of a bucket is one contiguous stretch. A
//      bucket of more than kTpSegment entries (a few heavy columns) is cut
//      into segments whose counts are summed in one kernel more, so one heavy
//      column does not serialise the sort.
// Values travel with their entries: nothing is gathered through a
// permutation. Larger matrices take the least-significant-digit radix sort
// below: 8-bit digits, ceil(bits(ncols - 1) / 8) passes, carrying each entry's
// position k in A:
//   1. per tile of kRxTile entries, a 256-bin digit histogram, stored
//      digit-major (hist[1 + d * ntiles + tile]);
//   2. an exclusive scan of those counts gives each (digit, tile) its first
//      output slot, so equal digits keep tile order;
//   3. each tile re-reads its entries in index order, ranks every entry
//      among equal digits before it (wavefront ballots on the 8 digit bits,
//      then per-wavefront counts in LDS) and scatters key and position.
// Then A^T's column indices are row(k), its values val[k], and its row
// pointer entry for column c is the first sorted position whose key is >= c
// (a binary search per column). Every step is deterministic: results do not
// depend on the order in which work-groups run.
//
// What bounds the two steps: about 60 bytes per float64 entry, 28 of them
// written, and the ranking's ballots. 128^3 convection-diffusion (14.6 M
// entries, 3 digits), one MI355X: 826 us by the radix sort (three scatters of
// 8-entry runs and a gather), 421 us now.
#include "convert.hpp"
#include "spmv_csr_tile.hpp"
#include "transpose.hpp"
#include "wave.hpp"

namespace spx {

constexpr int kRxThreads = 256;
constexpr int kRxItems = 8;
constexpr int kRxTile = kRxThreads * kRxItems;  // entries per work-group
constexpr int kRxBins = 256;
constexpr int kRxWaves = kRxThreads / kWave;

static int64_t rx_tiles(int64_t nnz) { return nnz > 0 ? ceil_div(nnz, kRxTile) : 1; }

// Radix passes needed for keys in [0, ncols).
static int rx_passes(int32_t ncols)
{
    int bits = 0;
    while (bits < 31 && (int64_t(1) << bits) < (int64_t)ncols) ++bits;
    return (bits + 7) / 8;
}

__global__ __launch_bounds__(kRxThreads) void rx_hist_kernel(const int32_t *__restrict__ keys, int64_t nnz, int shift,
                                                            int64_t ntiles, int32_t *__restrict__ hist)
{
    __shared__ int32_t h[kRxBins];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRxTile;
#pragma unroll
    for (int j = 0; j < kRxItems; ++j) {
        const int64_t e = base + j * kRxThreads + threadIdx.x;
        if (e < nnz) atomicAdd(&h[((uint32_t)keys[e] >> shift) & (kRxBins - 1)], 1);
    }
    __syncthreads();
    hist[1 + (int64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) hist[0] = 0;
}

// offs[d * ntiles + tile]: first output slot of digit d in this tile.
// perm_in == nullptr: the positions are the identity (first pass).
__global__ __launch_bounds__(kRxThreads) void rx_scatter_kernel(const int32_t *__restrict__ keys_in,
                                                               const int32_t *__restrict__ perm_in, int64_t nnz,
                                                               int shift, int64_t ntiles,
                                                               const int32_t *__restrict__ offs,
                                                               int32_t *__restrict__ keys_out,
                                                               int32_t *__restrict__ perm_out)
{
    __shared__ int32_t run[kRxBins];
    __shared__ int32_t cnt[kRxWaves][kRxBins];
    const int w = threadIdx.x / kWave;
    run[threadIdx.x] = offs[(int64_t)threadIdx.x * ntiles + blockIdx.x];
#pragma unroll
    for (int v = 0; v < kRxWaves; ++v) cnt[v][threadIdx.x] = 0;
    __syncthreads();
    const lane_mask_t below = (lane_mask_t(1) << lane_id()) - 1;
    const int64_t base = (int64_t)blockIdx.x * kRxTile;
    for (int j = 0; j < kRxItems; ++j) {
        const int64_t e = base + j * kRxThreads + threadIdx.x;
        const bool valid = e < nnz;
        const int32_t key = valid ? keys_in[e] : 0;
        const int d = (int)(((uint32_t)key >> shift) & (kRxBins - 1));
        // lanes of this wavefront holding the same digit
        lane_mask_t peers = ballot64(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1;
            const lane_mask_t m = ballot64(bit);
            peers &= bit ? m : ~m;
        }
        const int rank = __popcll(peers & below);
        const bool leader = valid && rank == 0;
        const int count = __popcll(peers);
        if (leader) cnt[w][d] = count;
        __syncthreads();
        if (valid) {
            int32_t pos = run[d] + rank;
            for (int v = 0; v < w; ++v) pos += cnt[v][d];
            keys_out[pos] = key;
            perm_out[pos] = perm_in ? perm_in[e] : (int32_t)e;
        }
        __syncthreads();
        // every read of run[] and cnt[] for this step is done; the next
        // step's writes to cnt[w][*] come from this same wavefront, in order
        if (leader) {
            atomicAdd(&run[d], count);
            cnt[w][d] = 0;
        }
    }
}

// rowptr_t[c] = first position p with keys[p] >= c (c = 0 .. ncols).
__global__ __launch_bounds__(kRxThreads) void rx_rowptr_kernel(const int32_t *__restrict__ keys, int64_t nnz,
                                                              int32_t ncols, int32_t *__restrict__ rowptr_t)
{
    const int64_t c = (int64_t)blockIdx.x * kRxThreads + threadIdx.x;
    if (c > ncols) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    rowptr_t[c] = (int32_t)lo;
}

// col_t[p] = row of entry perm[p], val_t[p] = val[perm[p]] (perm == nullptr:
// identity). T is an unsigned integer of the value's width (bit copy).
template <typename T>
__global__ __launch_bounds__(kRxThreads) void rx_gather_kernel(const int32_t *__restrict__ perm, int64_t nnz,
                                                              const int32_t *__restrict__ rowof,
                                                              const T *__restrict__ val, int32_t *__restrict__ col_t,
                                                              T *__restrict__ val_t)
{
    const int64_t p = (int64_t)blockIdx.x * kRxThreads + threadIdx.x;
    if (p >= nnz) return;
    const int32_t k = perm ? perm[p] : (int32_t)p;
    col_t[p] = rowof[k];
    val_t[p] = val[k];
}

struct RxBufs {
    int32_t *rowof, *k0, *k1, *p0, *p1, *hist;
    void *scan;
};

static RxBufs rx_carve(char *base, int64_t nnz, size_t *total)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = (off + 255) & ~size_t(255);
        char *p = base ? base + off : nullptr;
        off += bytes > 0 ? bytes : 1;
        return p;
    };
    const int64_t ntiles = rx_tiles(nnz);
    const size_t e = (size_t)(nnz > 0 ? nnz : 1) * sizeof(int32_t);
    RxBufs b;
    b.rowof = reinterpret_cast<int32_t *>(take(e));
    b.k0 = reinterpret_cast<int32_t *>(take(e));
    b.k1 = reinterpret_cast<int32_t *>(take(e));
    b.p0 = reinterpret_cast<int32_t *>(take(e));
    b.p1 = reinterpret_cast<int32_t *>(take(e));
    b.hist = reinterpret_cast<int32_t *>(take((size_t)(kRxBins * ntiles + 1) * sizeof(int32_t)));
    b.scan = take((size_t)scan_ws_bytes(kRxBins * ntiles));
    *total = off + 256;
    return b;
}

// ------------------------------------------------------------------ two-step sort
constexpr int kTpThreads = 256;
constexpr int kTpWaves = kTpThreads / kWave;
constexpr int kTpItems = 16;                      // entries per lane of the partition
constexpr int kTpWaveTile = kWave * kTpItems;     // entries per wavefront
constexpr int kTpTile = kTpWaves * kTpWaveTile;   // entries per work-group
constexpr int kTpMaxBuckets = 2048;
constexpr int kTpMaxWidth = 2048;                 // columns per bucket
constexpr int kTpGroups = 64;                     // groups of tiles in the prefix sums
constexpr int kTpSegment = 16384;                 // entries of a bucket per work-group
constexpr int kTpScanThreads = 1024;
constexpr int kTpSortThreads = 512;               // of the one-segment sort
constexpr int kTpSortWaves = kTpSortThreads / kWave;

// A wavefront walks the rows of its entries 64 at a time; where more than this
// many steps do not reach its last entry (runs of empty rows: fewer than one
// entry in two rows), it searches for every entry's row instead. 1,000 entries
// in 10 million rows: the transpose 47 ms walked, 93 us searched.
constexpr int kTpRowSteps = 32;
constexpr int kTpColBits = 22;
static_assert((int64_t)kTpMaxBuckets * kTpMaxWidth == int64_t(1) << kTpColBits, "a column fits its bits");
static_assert(kTpWaveTile <= 1 << (32 - kTpColBits), "and a wavefront's entries the rest");

struct TpShape {
    int32_t ncols, buckets;
    int shift;      // log2 columns per bucket
    int64_t tiles;
};

// Buckets of 2^shift columns: of at most kTpFill entries on average, so that
// few exceed a segment, and not fewer than 512 of them unless they would hold
// less than 2,048 entries. 0 buckets: more columns or entries than the two
// steps take.
constexpr int64_t kTpFill = kTpSegment * 9 / 10;

static TpShape tp_shape(int32_t ncols, int64_t nnz)
{
    TpShape t{ncols, 0, 0, ceil_div(nnz, kTpTile)};
    if (ncols > kTpMaxBuckets * kTpMaxWidth || nnz > kTpMaxBuckets * kTpFill) return t;
    int64_t fill = nnz / 512;
    fill = fill < 2048 ? 2048 : (fill > kTpFill ? kTpFill : fill);
    int64_t want = ceil_div(nnz, fill);  // buckets
    if (want > kTpMaxBuckets) want = kTpMaxBuckets;
    // the widest buckets that are at least so many (or one column each)
    while ((2 << t.shift) <= kTpMaxWidth && ceil_div(ncols, int64_t(2) << t.shift) >= want) ++t.shift;
    while (ceil_div(ncols, int64_t(1) << t.shift) > kTpMaxBuckets) ++t.shift;
    t.buckets = (int32_t)ceil_div(ncols, int64_t(1) << t.shift);
    return t;
}

// Columns outside [0, ncols) sort as the last one: wrong input gives a wrong
// result, not a wild access.
__device__ __forceinline__ uint32_t tp_key(int32_t c, int32_t ncols)
{
    return (uint32_t)c < (uint32_t)ncols ? (uint32_t)c : (uint32_t)ncols - 1u;
}

// Lanes (of those in `valid`) that hold the same key of `bits` <= 11 bits as
// this one.
__device__ __forceinline__ lane_mask_t tp_peers(uint32_t key, int bits, bool valid)
{
    const lane_mask_t all = ballot64(valid);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
    for (int b = 0; b < bits; ++b) {
        const uint32_t other = ((key >> b) & 1u) - 1u;  // all ones where the bit is clear
        const lane_mask_t m = ballot64(other == 0u);
        lo &= (uint32_t)m ^ other;
        hi &= (uint32_t)(m >> 32) ^ other;
    }
    return ((lane_mask_t)hi << 32) | lo;
}

// hist[tile * buckets + b]: entries of the tile in bucket b.
__global__ __launch_bounds__(kTpThreads) void tp_hist_kernel(const int32_t *__restrict__ col, int64_t nnz,
                                                            int32_t ncols, int shift, int32_t buckets,
                                                            int32_t *__restrict__ hist)
{
    __shared__ int32_t h[kTpMaxBuckets];
    for (int b = threadIdx.x; b < buckets; b += kTpThreads) h[b] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kTpTile;
    int32_t key[kTpTile / kTpThreads];
#pragma unroll
    for (int j = 0; j < kTpTile / kTpThreads; ++j) {
        const int64_t e = base + j * kTpThreads + threadIdx.x;
        key[j] = e < nnz ? (int32_t)(tp_key(col[e], ncols) >> shift) : -1;
    }
#pragma unroll
    for (int j = 0; j < kTpTile / kTpThreads; ++j) {
        // banded rows put a wavefront's 64 entries into a few buckets: up to
        // eight of them are counted with one add each, not 64 adds to few words
        lane_mask_t left = ballot64(key[j] >= 0);
        for (int it = 0; it < 8 && left != 0; ++it) {
            const int32_t k = readlane(key[j], __builtin_ctzll(left));
            const lane_mask_t m = ballot64(key[j] == k);
            if (__popcll(m) < 4) break;  // scattered
            if (lane_id() == 0) atomicAdd(&h[k], __popcll(m));
            left &= ~m;
        }
        if ((left >> lane_id()) & 1) atomicAdd(&h[key[j]], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < buckets; b += kTpThreads) hist[(int64_t)blockIdx.x * buckets + b] = h[b];
}

// Sums of hist over each group of `per` tiles (work-group: one group).
__global__ __launch_bounds__(kTpScanThreads) void tp_group_sums(const int32_t *__restrict__ hist, int64_t tiles,
                                                               int64_t per, int32_t buckets,
                                                               int32_t *__restrict__ gsum)
{
    const int64_t t0 = blockIdx.x * per, t1 = t0 + per < tiles ? t0 + per : tiles;
    for (int b = threadIdx.x; b < buckets; b += kTpScanThreads) {
        int32_t s = 0;
#pragma unroll 8
        for (int64_t t = t0; t < t1; ++t) s += hist[t * buckets + b];
        gsum[(int64_t)blockIdx.x * buckets + b] = s;
    }
}

// Exclusive sum of v over the work-group's threads (kThreads of them).
template <int kThreads>
__device__ __forceinline__ int32_t tp_block_exclusive(int32_t v, int32_t *s_wave)
{
    int32_t inc = v;
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t o = __shfl_up(inc, off);
        if (lane_id() >= off) inc += o;
    }
    if (lane_id() == kWave - 1) s_wave[threadIdx.x / kWave] = inc;
    __syncthreads();
    int32_t before = 0;
    for (int w = 0; w < (int)threadIdx.x / kWave; ++w) before += s_wave[w];
    __syncthreads();
    return before + inc - v;
}

// Bucket starts, the segments of every bucket (segstart) and those of the
// buckets that have several (multistart); gsum[g][b] becomes the first slot of
// group g's entries of bucket b. One work-group, kPer buckets a thread.
template <int kPer>
__global__ __launch_bounds__(kTpScanThreads) void tp_bucket_scan(int32_t *__restrict__ gsum, int groups,
                                                                int32_t buckets, int32_t *__restrict__ bstart,
                                                                int32_t *__restrict__ segstart,
                                                                int32_t *__restrict__ multistart)
{
    __shared__ int32_t s_wave[kTpScanThreads / kWave];
    int32_t tot[kPer], seg[kPer], multi[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int b = threadIdx.x * kPer + u;
        tot[u] = seg[u] = multi[u] = 0;
        if (b < buckets) {
#pragma unroll 8
            for (int g = 0; g < groups; ++g) tot[u] += gsum[(int64_t)g * buckets + b];
            seg[u] = tot[u] > kTpSegment ? (tot[u] - 1) / kTpSegment + 1 : 1;
            multi[u] = seg[u] > 1 ? seg[u] : 0;
        }
    }
    int32_t tt = 0, ss = 0, mm = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        tt += tot[u];
        ss += seg[u];
        mm += multi[u];
    }
    int32_t b0 = tp_block_exclusive<kTpScanThreads>(tt, s_wave);
    int32_t s0 = tp_block_exclusive<kTpScanThreads>(ss, s_wave);
    int32_t m0 = tp_block_exclusive<kTpScanThreads>(mm, s_wave);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int b = threadIdx.x * kPer + u;
        if (b < buckets) {
            bstart[b] = b0;
            segstart[b] = s0;
            multistart[b] = m0;
            int32_t run = b0;
#pragma unroll 8
            for (int g = 0; g < groups; ++g) {
                const int32_t t = gsum[(int64_t)g * buckets + b];
                gsum[(int64_t)g * buckets + b] = run;
                run += t;
            }
        }
        b0 += tot[u];
        s0 += seg[u];
        m0 += multi[u];
        if (b == buckets - 1) {
            bstart[buckets] = b0;
            segstart[buckets] = s0;
            multistart[buckets] = m0;
        }
    }
}

// hist[tile][b] becomes the first slot of the tile's entries of bucket b.
__global__ __launch_bounds__(kTpScanThreads) void tp_tile_offsets(int32_t *__restrict__ hist, int64_t tiles,
                                                                 int64_t per, int32_t buckets,
                                                                 const int32_t *__restrict__ gsum)
{
    const int64_t t0 = blockIdx.x * per, t1 = t0 + per < tiles ? t0 + per : tiles;
    for (int b = threadIdx.x; b < buckets; b += kTpScanThreads) {
        int32_t run = gsum[(int64_t)blockIdx.x * buckets + b];
#pragma unroll 8
        for (int64_t t = t0; t < t1; ++t) {
            const int32_t v = hist[t * buckets + b];
            hist[t * buckets + b] = run;
            run += v;
        }
    }
}

// Inclusive maximum over the lanes of a wavefront (values >= -1).
__device__ __forceinline__ int32_t tp_scan_max(int32_t v)
{
    auto up = [](int32_t a, int32_t b) { return a > b ? a : b; };
    v = up(v, dpp<0x111>(-1, v));
    v = up(v, dpp<0x112>(-1, v));
    v = up(v, dpp<0x114>(-1, v));
    v = up(v, dpp<0x118>(-1, v));
    v = up(v, dpp<kRowBcast15, 0xA>(-1, v));
    v = up(v, dpp<kRowBcast31, 0xC>(-1, v));
    return v;
}

// The row of every entry of [e0, e1), each by its own bisection of
// [first, nrows] (the last row that starts at or before it): all of a lane's
// entries step by step together, so that a step costs one load's latency.
__device__ void tp_find_rows(const int32_t *__restrict__ rowptr, int64_t first, int32_t nrows, int64_t e0, int64_t e1,
                             int32_t *__restrict__ s_row)
{
    int32_t at[kTpItems];
#pragma unroll
    for (int u = 0; u < kTpItems; ++u) at[u] = (int32_t)first;
    int64_t step = 1;
    while (first + step < nrows) step *= 2;
    for (; step > 0; step /= 2) {
#pragma unroll
        for (int u = 0; u < kTpItems; ++u) {
            const int64_t e = e0 + u * kWave + lane_id(), r = at[u] + step;
            if (r < nrows && e < e1 && rowptr[r] <= e) at[u] = (int32_t)r;
        }
    }
#pragma unroll
    for (int u = 0; u < kTpItems; ++u) s_row[u * kWave + lane_id()] = at[u];
}

// Entries to their buckets, in order. T: unsigned integer of the value's width.
template <typename T>
__global__ __launch_bounds__(kTpThreads) void tp_partition_kernel(
    const int32_t *__restrict__ rowptr, int32_t nrows, const int32_t *__restrict__ col, const T *__restrict__ val,
    int64_t nnz, int32_t ncols, int shift, int bits, int32_t buckets, const int32_t *__restrict__ offs,
    int32_t *__restrict__ col_out, int32_t *__restrict__ row_out, T *__restrict__ val_out)
{
    extern __shared__ int32_t s_cnt[];  // [kTpWaves][buckets]
    __shared__ int32_t s_row[kTpWaves][kTpWaveTile];
    // neighbouring tiles on one XCD: their entries of a bucket are neighbours
    // in the output, and meet in its L2
    const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
    if (tile * kTpTile >= nnz) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    int32_t *cnt = s_cnt + w * buckets;
    for (int b = threadIdx.x; b < kTpWaves * buckets; b += kTpThreads) s_cnt[b] = 0;
    for (int i = lane; i < kTpWaveTile; i += kWave) s_row[w][i] = -1;
    __syncthreads();
    const int64_t e0 = tile * kTpTile + (int64_t)w * kTpWaveTile;
    const int64_t e1 = e0 + kTpWaveTile < nnz ? e0 + kTpWaveTile : nnz;
    uint32_t c[kTpItems];  // column, and above kTpColBits the place among the wavefront's entries of its bucket
#pragma unroll
    for (int u = 0; u < kTpItems; ++u) {
        const int64_t e = e0 + u * kWave + lane;
        c[u] = e < e1 ? tp_key(col[e], ncols) : 0u;
    }
    if (e0 < e1) {
        // mark where this stretch's rows start (of several rows that start at
        // one entry the last is the one that holds it)
        int32_t v;
        const int64_t first = lower_bound_wave(rowptr, 0, nrows, e0 + 1, &v) - 1;
        int64_t r = first + lane;
        bool walked = false;
        for (int step = 0; step < kTpRowSteps && !walked; ++step, r += kWave) {
            const int64_t start = r < nrows ? rowptr[r] : e1;
            if (start < e1) atomicMax(&s_row[w][start > e0 ? start - e0 : 0], (int32_t)r);
            walked = ballot64(start >= e1) != 0;
        }
        if (!walked) tp_find_rows(rowptr, first, nrows, e0, e1, s_row[w]);
    }
    const lane_mask_t below = (lane_mask_t(1) << lane) - 1;
#pragma unroll
    for (int u = 0; u < kTpItems; ++u) {
        const bool valid = e0 + u * kWave + lane < e1;
        const uint32_t b = c[u] >> shift;
        const lane_mask_t peers = tp_peers(b, bits, valid);
        const int rank = __popcll(peers & below);
        const int32_t first = cnt[b];
        if (valid && rank == 0) cnt[b] = first + __popcll(peers);  // this wavefront's own counter
        c[u] |= (uint32_t)(first + rank) << kTpColBits;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    for (int b = threadIdx.x; b < buckets; b += kTpThreads) {
        int32_t run = offs[tile * buckets + b];
#pragma unroll
        for (int q = 0; q < kTpWaves; ++q) {
            const int32_t t = s_cnt[q * buckets + b];
            s_cnt[q * buckets + b] = run;
            run += t;
        }
    }
    __syncthreads();
    int32_t row_before = -1;
#pragma unroll
    for (int u = 0; u < kTpItems; ++u) {
        const int64_t e = e0 + u * kWave + lane;
        const bool valid = e < e1;
        const T x = valid ? val[e] : T(0);
        int32_t row = tp_scan_max(s_row[w][u * kWave + lane]);
        row = row > row_before ? row : row_before;
        row_before = readlane(row, kWave - 1);
        const uint32_t column = c[u] & ((1u << kTpColBits) - 1);
        if (valid) {
            const int32_t pos = cnt[column >> shift] + (int32_t)(c[u] >> kTpColBits);
            col_out[pos] = (int32_t)column;
            row_out[pos] = row;
            val_out[pos] = x;
        }
    }
}

// The bucket and the segment of it that work-group g takes; false: none.
__device__ __forceinline__ bool tp_segment(int32_t g, int32_t buckets, const int32_t *__restrict__ segstart,
                                           int32_t *bucket, int32_t *seg, bool *multi)
{
    if (g >= segstart[buckets]) return false;
    int32_t lo = 0, hi = buckets;  // segstart[lo] <= g < segstart[hi]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (segstart[mid] <= g) lo = mid;
        else hi = mid;
    }
    *bucket = lo;
    *seg = g - segstart[lo];
    *multi = segstart[lo + 1] - segstart[lo] > 1;
    return true;
}

// Buckets of one segment, one work-group each: counts per column and
// wavefront, their scan (and A^T's row pointer), then the entries' places:
// the sorted order is formed in LDS and the output written in order, gathering
// the entries (of a banded matrix a few runs) rather than scattering them
// over the bucket's 170 KB, of which a whole XCD's do not fit its L2.
template <typename T>
__global__ __launch_bounds__(kTpSortThreads) void tp_bucket_kernel(
    const int32_t *__restrict__ col_in, const int32_t *__restrict__ row_in, const T *__restrict__ val_in,
    int32_t ncols, int shift, int32_t buckets, const int32_t *__restrict__ bstart,
    const int32_t *__restrict__ segstart, int32_t *__restrict__ rowptr_t, int32_t *__restrict__ col_t,
    T *__restrict__ val_t)
{
    extern __shared__ uint32_t s_cnt2[];  // [kTpSortWaves][width] 16-bit counts, two to a word
    __shared__ uint16_t s_from[kTpSegment];
    __shared__ int32_t s_wave[kTpSortWaves];
    int32_t bucket, seg;
    bool multi;
    if (!tp_segment((int32_t)blockIdx.x, buckets, segstart, &bucket, &seg, &multi) || multi) return;
    uint16_t *s_cnt = reinterpret_cast<uint16_t *>(s_cnt2);
    const int width = 1 << shift, mask = width - 1;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    // counts are kept column by column: [column][wavefront]
    for (int c = threadIdx.x; c < kTpSortWaves * width / 2; c += kTpSortThreads) s_cnt2[c] = 0u;
    __syncthreads();
    const int64_t p0 = bstart[bucket];
    const int n = (int)(bstart[bucket + 1] - p0);
    const int32_t *__restrict__ cols = col_in + p0;
    // each wavefront takes a contiguous share, in chunks of 64: an entry's
    // column, and above 16 bits its place among the share's entries of it
    const int share = ((n + kTpSortThreads - 1) / kTpSortThreads) * kWave;
    const int q0 = w * share < n ? w * share : n;
    const int q1 = q0 + share < n ? q0 + share : n;
    constexpr int kChunks = kTpSegment / kTpSortThreads;
    const lane_mask_t below = (lane_mask_t(1) << lane) - 1;
    uint32_t c[kChunks];
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
        const int e = q0 + u * kWave + lane;
        c[u] = e < q1 ? (uint32_t)(cols[e] & mask) : 0u;
    }
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
        if (q0 + u * kWave < q1) {  // uniform
            const bool valid = q0 + u * kWave + lane < q1;
            const lane_mask_t peers = tp_peers(c[u], shift, valid);
            const int rank = __popcll(peers & below);
            const int i = (int)c[u] * kTpSortWaves + w;
            const int first = s_cnt[i];
            if (valid && rank == 0) s_cnt[i] = (uint16_t)(first + __popcll(peers));  // this wavefront's own counter
            c[u] |= (uint32_t)(first + rank) << 16;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    __syncthreads();
    {
        // first slot of every (column, wavefront), a thread's columns in a row
        const int per = (width + kTpSortThreads - 1) / kTpSortThreads;
        const int c0 = (int)threadIdx.x * per < width ? (int)threadIdx.x * per : width;
        const int c1 = c0 + per < width ? c0 + per : width;
        int32_t t = 0;
        for (int i = c0 * kTpSortWaves; i < c1 * kTpSortWaves; ++i) t += s_cnt[i];
        int32_t run = tp_block_exclusive<kTpSortThreads>(t, s_wave);
        for (int k = c0; k < c1; ++k) {
            const int64_t column = ((int64_t)bucket << shift) + k;
            if (column < ncols) rowptr_t[column] = (int32_t)p0 + run;
            for (int i = k * kTpSortWaves; i < (k + 1) * kTpSortWaves; ++i) {
                const int32_t v = s_cnt[i];
                s_cnt[i] = (uint16_t)run;
                run += v;
            }
        }
        if (bucket == buckets - 1 && threadIdx.x == 0) rowptr_t[ncols] = (int32_t)p0 + n;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
        const int e = q0 + u * kWave + lane;
        if (e < q1) s_from[s_cnt[(c[u] & 0xffffu) * kTpSortWaves + w] + (c[u] >> 16)] = (uint16_t)e;
    }
    __syncthreads();
#pragma unroll 8
    for (int o = threadIdx.x; o < n; o += kTpSortThreads) {
        const int e = s_from[o];
        col_t[p0 + o] = row_in[p0 + e];
        val_t[p0 + o] = val_in[p0 + e];
    }
}

// One work-group per segment of the buckets that have several. kSort = false:
// the segment's counts per column; true, once tp_multi_scan has turned these
// into first slots: the sort.
template <typename T, bool kSort>
__global__ __launch_bounds__(kTpThreads) void tp_multi_kernel(
    const int32_t *__restrict__ col_in, const int32_t *__restrict__ row_in, const T *__restrict__ val_in, int shift,
    int32_t buckets, const int32_t *__restrict__ bstart, const int32_t *__restrict__ segstart,
    const int32_t *__restrict__ multistart, int32_t *__restrict__ segcnt, int32_t *__restrict__ col_t,
    T *__restrict__ val_t)
{
    extern __shared__ int32_t s_cnt4[];  // [kTpWaves][1 << shift]
    int32_t bucket, seg;
    bool multi;
    if (!tp_segment((int32_t)blockIdx.x, buckets, segstart, &bucket, &seg, &multi) || !multi) return;
    const int width = 1 << shift, mask = width - 1;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    int32_t *cnt = s_cnt4 + w * width;
    for (int c = threadIdx.x; c < kTpWaves * width; c += kTpThreads) s_cnt4[c] = 0;
    __syncthreads();
    const int64_t p0 = bstart[bucket] + (int64_t)seg * kTpSegment, pe = bstart[bucket + 1];
    const int64_t p1 = p0 + kTpSegment < pe ? p0 + kTpSegment : pe;
    // each wavefront takes a contiguous quarter
    const int64_t quarter = ((p1 - p0 + kTpThreads - 1) / kTpThreads) * kWave;
    const int64_t q0 = p0 + w * quarter < p1 ? p0 + w * quarter : p1;
    const int64_t q1 = q0 + quarter < p1 ? q0 + quarter : p1;
#pragma unroll 8
    for (int64_t e = q0 + lane; e < q1; e += kWave) atomicAdd(&cnt[col_in[e] & mask], 1);
    __syncthreads();
    int32_t *first_of = segcnt + (int64_t)(multistart[bucket] + seg) * width;
    for (int c = threadIdx.x; c < width; c += kTpThreads) {
        int32_t run = kSort ? first_of[c] : 0;
        for (int q = 0; q < kTpWaves; ++q) {
            const int32_t v = s_cnt4[q * width + c];
            s_cnt4[q * width + c] = run;
            run += v;
        }
        if (!kSort) first_of[c] = run;
    }
    if (!kSort) return;
    __syncthreads();
    const lane_mask_t below = (lane_mask_t(1) << lane) - 1;
    constexpr int kU = 4;  // chunks in flight
    for (int64_t e0 = q0; e0 < q1; e0 += kU * kWave) {
        int32_t c[kU], r[kU];
        T x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t e = e0 + u * kWave + lane;
            const bool valid = e < q1;
            c[u] = valid ? col_in[e] & mask : 0;
            r[u] = valid ? row_in[e] : 0;
            x[u] = valid ? val_in[e] : T(0);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const bool valid = e0 + u * kWave + lane < q1;
            const lane_mask_t peers = tp_peers((uint32_t)c[u], shift, valid);
            const int rank = __popcll(peers & below);
            const int32_t first = cnt[c[u]];
            if (valid) {
                if (rank == 0) cnt[c[u]] = first + __popcll(peers);  // this wavefront's own counter
                col_t[first + rank] = r[u];
                val_t[first + rank] = x[u];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
}

// Buckets of several segments: counts per segment and column to first slots,
// and A^T's row pointer.
__global__ __launch_bounds__(kTpThreads) void tp_multi_scan(int32_t ncols, int shift, int32_t buckets,
                                                           const int32_t *__restrict__ bstart,
                                                           const int32_t *__restrict__ multistart,
                                                           int32_t *__restrict__ segcnt,
                                                           int32_t *__restrict__ rowptr_t)
{
    __shared__ int32_t s_wave[kTpWaves];
    const int32_t bucket = (int32_t)blockIdx.x;
    const int32_t m0 = multistart[bucket], m1 = multistart[bucket + 1];
    if (m0 == m1) return;
    const int width = 1 << shift;
    const int per = (width + kTpThreads - 1) / kTpThreads;
    const int c0 = (int)threadIdx.x * per, c1 = c0 + per < width ? c0 + per : width;
    int32_t t = 0;
    for (int c = c0; c < c1; ++c)
#pragma unroll 8
        for (int32_t m = m0; m < m1; ++m) t += segcnt[(int64_t)m * width + c];
    int32_t run = bstart[bucket] + tp_block_exclusive<kTpThreads>(t, s_wave);
    for (int c = c0; c < c1; ++c) {
        const int64_t column = ((int64_t)bucket << shift) + c;
        if (column < ncols) rowptr_t[column] = run;
        for (int32_t m = m0; m < m1; ++m) {
            const int32_t v = segcnt[(int64_t)m * width + c];
            segcnt[(int64_t)m * width + c] = run;
            run += v;
        }
    }
    if (bucket == buckets - 1 && threadIdx.x == 0) rowptr_t[ncols] = bstart[buckets];
}

struct TpBufs {
    int32_t *col, *row, *hist, *gsum, *bstart, *segstart, *multistart, *segcnt;
    void *val;
};

// For any number of columns that the sort takes (sized by nnz alone).
static TpBufs tp_carve(char *base, int64_t nnz, size_t *total)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = (off + 255) & ~size_t(255);
        char *p = base ? base + off : nullptr;
        off += bytes > 0 ? bytes : 1;
        return p;
    };
    const int64_t tiles = ceil_div(nnz, kTpTile);
    TpBufs b;
    b.val = take((size_t)nnz * 8);
    b.col = reinterpret_cast<int32_t *>(take((size_t)nnz * 4));
    b.row = reinterpret_cast<int32_t *>(take((size_t)nnz * 4));
    b.hist = reinterpret_cast<int32_t *>(take((size_t)tiles * kTpMaxBuckets * 4));
    b.gsum = reinterpret_cast<int32_t *>(take((size_t)(tiles < kTpGroups ? tiles : kTpGroups) * kTpMaxBuckets * 4));
    b.bstart = reinterpret_cast<int32_t *>(take((kTpMaxBuckets + 1) * 4));
    b.segstart = reinterpret_cast<int32_t *>(take((kTpMaxBuckets + 1) * 4));
    b.multistart = reinterpret_cast<int32_t *>(take((kTpMaxBuckets + 1) * 4));
    // a bucket of several segments holds more than kTpSegment entries: at
    // most 2 nnz / kTpSegment such segments
    b.segcnt = reinterpret_cast<int32_t *>(take((size_t)(2 * nnz / kTpSegment) * kTpMaxWidth * 4));
    *total = off + 256;
    return b;
}

template <typename T>
static spx_status tp_run(const spx_matrix &A, spx_matrix &At, const TpShape &t, const TpBufs &b, hipStream_t stream)
{
    const int64_t nnz = A.nnz;
    const T *val = static_cast<const T *>(A.vals);
    T *bval = static_cast<T *>(b.val), *val_t = static_cast<T *>(At.vals);
    const int64_t groups = t.tiles < kTpGroups ? t.tiles : kTpGroups;
    const int64_t per = ceil_div(t.tiles, groups);
    int bits = 0;
    while ((1 << bits) < t.buckets) ++bits;
    tp_hist_kernel<<<(unsigned)t.tiles, kTpThreads, 0, stream>>>(A.colidx, nnz, t.ncols, t.shift, t.buckets, b.hist);
    int32_t *gsum = per > 1 ? b.gsum : b.hist;  // groups of one tile: their sums are its counts
    if (per > 1)
        tp_group_sums<<<(unsigned)groups, kTpScanThreads, 0, stream>>>(b.hist, t.tiles, per, t.buckets, gsum);
    if (t.buckets <= kTpScanThreads)
        tp_bucket_scan<1><<<1, kTpScanThreads, 0, stream>>>(gsum, (int)groups, t.buckets, b.bstart, b.segstart,
                                                            b.multistart);
    else
        tp_bucket_scan<2><<<1, kTpScanThreads, 0, stream>>>(gsum, (int)groups, t.buckets, b.bstart, b.segstart,
                                                            b.multistart);
    if (per > 1)
        tp_tile_offsets<<<(unsigned)groups, kTpScanThreads, 0, stream>>>(b.hist, t.tiles, per, t.buckets, gsum);
    const size_t lds_p = (size_t)kTpWaves * t.buckets * 4, lds_b = (size_t)kTpWaves * ((size_t)4 << t.shift);
    const size_t lds_s = (size_t)kTpSortWaves * ((size_t)2 << t.shift);
    tp_partition_kernel<T><<<(unsigned)pad_to_xcds(t.tiles), kTpThreads, lds_p, stream>>>(
        A.rowptr, A.nrows, A.colidx, val, nnz, t.ncols, t.shift, bits, t.buckets, b.hist, b.col, b.row, bval);
    SPX_LAUNCHED();
    const unsigned segs = (unsigned)(t.buckets + nnz / kTpSegment);
    tp_bucket_kernel<T><<<segs, kTpSortThreads, lds_s, stream>>>(b.col, b.row, bval, t.ncols, t.shift, t.buckets,
                                                                b.bstart, b.segstart, At.rowptr, At.colidx, val_t);
    if (nnz > kTpSegment) {  // else no bucket has several segments
        tp_multi_kernel<T, false><<<segs, kTpThreads, lds_b, stream>>>(b.col, b.row, bval, t.shift, t.buckets,
                                                                      b.bstart, b.segstart, b.multistart, b.segcnt,
                                                                      At.colidx, val_t);
        tp_multi_scan<<<(unsigned)t.buckets, kTpThreads, 0, stream>>>(t.ncols, t.shift, t.buckets, b.bstart,
                                                                     b.multistart, b.segcnt, At.rowptr);
        tp_multi_kernel<T, true><<<segs, kTpThreads, lds_b, stream>>>(b.col, b.row, bval, t.shift, t.buckets,
                                                                     b.bstart, b.segstart, b.multistart, b.segcnt,
                                                                     At.colidx, val_t);
    }
    SPX_LAUNCHED();
    return SPX_OK;
}

int64_t transpose_ws_bytes(int64_t nnz)
{
    size_t rx = 0, tp = 0;
    (void)rx_carve(nullptr, nnz, &rx);
    (void)tp_carve(nullptr, nnz, &tp);
    return (int64_t)(rx > tp ? rx : tp);
}

spx_status transpose_run(const spx_matrix &A, spx_matrix &At, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const int64_t nnz = A.nnz;
    const int32_t ncols = (int32_t)A.ncols;
    const size_t need = (size_t)transpose_ws_bytes(nnz);
    SPX_REQUIRE(ws != nullptr && ws_bytes >= need, SPX_ERR_ARG,
                "csr transpose: workspace of %zu bytes is too small (need %zu)", ws_bytes, need);
    // round the base up to 256 bytes inside the slack the size includes
    char *base = reinterpret_cast<char *>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
    size_t total = 0;
    const TpShape t = tp_shape(ncols, nnz);
    if (nnz > 0 && t.buckets > 0) {
        const TpBufs tb = tp_carve(base, nnz, &total);
        switch (A.val_type) {
        case SPX_F64: return tp_run<uint64_t>(A, At, t, tb, stream);
        case SPX_F32: return tp_run<uint32_t>(A, At, t, tb, stream);
        default: return tp_run<uint16_t>(A, At, t, tb, stream);
        }
    }
    RxBufs b = rx_carve(base, nnz, &total);
    const unsigned grow = (unsigned)ceil_div((int64_t)ncols + 1, kRxThreads);
    if (nnz == 0) {
        rx_rowptr_kernel<<<grow, kRxThreads, 0, stream>>>(b.k0, 0, ncols, At.rowptr);
        SPX_LAUNCHED();
        return SPX_OK;
    }
    SPX_CHECK(csr_rows_launch(A.rowptr, (int32_t)A.nrows, b.rowof, stream));
    const int64_t ntiles = rx_tiles(nnz);
    const int passes = rx_passes(ncols);
    const int32_t *keys = A.colidx;
    const int32_t *perm = nullptr;
    int32_t *kout = b.k0, *pout = b.p0;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        rx_hist_kernel<<<(unsigned)ntiles, kRxThreads, 0, stream>>>(keys, nnz, shift, ntiles, b.hist);
        SPX_LAUNCHED();
        SPX_CHECK(inclusive_scan<int32_t>(b.hist + 1, kRxBins * ntiles, b.scan, stream));
        rx_scatter_kernel<<<(unsigned)ntiles, kRxThreads, 0, stream>>>(keys, perm, nnz, shift, ntiles, b.hist, kout,
                                                                       pout);
        SPX_LAUNCHED();
        keys = kout;
        perm = pout;
        kout = (kout == b.k0) ? b.k1 : b.k0;
        pout = (pout == b.p0) ? b.p1 : b.p0;
    }
    rx_rowptr_kernel<<<grow, kRxThreads, 0, stream>>>(keys, nnz, ncols, At.rowptr);
    SPX_LAUNCHED();
    const unsigned g = (unsigned)ceil_div(nnz, kRxThreads);
    switch (A.val_type) {
    case SPX_F64:
        rx_gather_kernel<uint64_t><<<g, kRxThreads, 0, stream>>>(perm, nnz, b.rowof,
                                                                 static_cast<const uint64_t *>(A.vals), At.colidx,
                                                                 static_cast<uint64_t *>(At.vals));
        break;
    case SPX_F32:
        rx_gather_kernel<uint32_t><<<g, kRxThreads, 0, stream>>>(perm, nnz, b.rowof,
                                                                 static_cast<const uint32_t *>(A.vals), At.colidx,
                                                                 static_cast<uint32_t *>(At.vals));
        break;
    default:
        rx_gather_kernel<uint16_t><<<g, kRxThreads, 0, stream>>>(perm, nnz, b.rowof,
                                                                 static_cast<const uint16_t *>(A.vals), At.colidx,
                                                                 static_cast<uint16_t *>(At.vals));
        break;
    }
    SPX_LAUNCHED();
    return SPX_OK;
}

}  // namespace spx
