// batch_wide.hip -- CG on many large systems at once, several work-groups per
// system, no synchronisation between work-groups inside a launch.
//
// Unpreconditioned CG from x0 = 0 in the single-reduction form of Chronopoulos
// and Gear (1989): besides r and p the recurrences carry w = A r and
// s = A p, so both inner products of a step (r.r and r.w) come from one
// pass and a step needs one grid-wide synchronisation fewer than the
// Hestenes-Stiefel order (the same Krylov iterates in exact arithmetic).
// One iteration is two grid-wide phases over every listed system (a launch
// boundary is the only global synchronisation):
//   A  w = A r (or w = A x in the true-residual mode), partial sums of r.w:
//      the load-balanced CSR tile kernel over every listed system's tiles, or
//      its staged-rows form where the system's rows are short and even;
//   V  gamma = r.r and delta = r.w from the partials; beta = gamma / gamma_old,
//      alpha = gamma / (delta - beta gamma / alpha_old) (beta = 0 and
//      alpha = gamma / delta when the recurrences start); p = r + beta p,
//      s = w + beta s, x += alpha p, r -= alpha s, partial sums of the new
//      r.r (true-residual mode: r = b - w; init: r = b). The first block of
//      each system commits its scalar state into the other of two state
//      buffers.
// The step is taken only while r.r is above the tolerance; below it the
// system checks its true residual (one product of x) and either finishes or
// restarts the recurrences from it.
// Nonsymmetric systems run unpreconditioned BiCGSTAB (van der Vorst 1992, in
// the order of the one-work-group kernel) on the same two kernels, one step
// as three product + vector pairs (bphase 0: v = A p with r_hat.v partials,
// then alpha and s = r - alpha v with s.s partials; bphase 1: t = A s with
// t.s and t.t partials, then omega, x and r = s - omega t with r.r and
// r_hat.r partials; bphase 2: no product, then beta and the new p). A small
// ||s|| or ||r|| is confirmed with the true residual, whose sum is read by
// one more pair (bphase 3), which also starts the recurrences after init.
// Every work-group that needs a sum forms it from the same partials in the
// same order, so all of them take the same decisions. A system's virtual
// blocks, partials and summation order depend only on its own size; its
// arithmetic is therefore independent of the other systems in the launch.
#include "batch_cg.hpp"
#include "spmv_csr.hpp"
#include "spmv_csr_stage.hpp"
#include "spmv_csr_tile.hpp"
#include "wave.hpp"

namespace spx {

constexpr int kWideWaves = kWideThreads / kWave;
constexpr int kWideStageWaves = kCsrThreads / kWave;
constexpr int kWideStageCap = 512;   // entries a wavefront stages at once
constexpr int kWideStageForms = 5;   // rows of up to 8, 16, 32, 64, 128 entries
static_assert(kWideThreads == kCsrThreads, "both phases reduce with the same work-group");

// kBytes per lane into LDS; see lds_copy16. Temporal: the solved systems'
// matrices are read again every iteration and may stay in the Infinity Cache.
template <int kBytes>
__device__ __forceinline__ void wide_copy(const void *g, void *lds)
{
    auto *from = (__attribute__((address_space(1))) const void *)g;
    auto *to = (__attribute__((address_space(3))) void *)lds;
    if constexpr (kBytes == 16) __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
    else __builtin_amdgcn_global_load_lds(from, to, 4, 0, 0);
}

// Work-group sum in a fixed order (result in every thread).
__device__ __forceinline__ double wide_wg_sum(double v, double *s_red)
{
    v = wave_sum(v);
    __syncthreads();  // s_red may still be read by a previous call
    if (lane_id() == 0) s_red[threadIdx.x / kWave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWideWaves; ++w) t += s_red[w];
    return t;
}

// Sum of part[0..cnt): thread t takes t, t + 256, ... in order (eight
// strides' loads in flight), then the fixed work-group reduction.
__device__ __forceinline__ double wide_part_sum(const double *part, int32_t cnt, double *s_red)
{
    double t = 0.0;
#pragma unroll 8
    for (int32_t i = threadIdx.x; i < cnt; i += kWideThreads) t += part[i];
    return wide_wg_sum(t, s_red);
}

// Row-length test of the staged product, spread over the blocks of the init
// phase: the longest row of rows [r0, r1) (result in thread 0).
__device__ double wide_longest_row(const WideSlot &S, int32_t r0, int32_t r1, double *s_red)
{
    int32_t m = 0;
    for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) m = max(m, S.rowptr[i + 1] - S.rowptr[i]);
#pragma unroll
    for (int d = kWave / 2; d > 0; d /= 2) m = max(m, __shfl_xor(m, d));
    __syncthreads();
    if (lane_id() == 0) s_red[threadIdx.x / kWave] = (double)m;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWideWaves; ++w) t = fmax(t, s_red[w]);
    return t;
}

// Product form of a system from its blocks' longest rows: the rule of the
// single product's staged-rows kernel, but for the arrays' alignment: a
// system's bits must not depend on where its arrays lie. len is the power of two at or above
// the longest row; rows fill at least half of len on average, so that the
// ceil(n * len / 4096) row blocks are never more than the ntiles tiles.
// Returns 1 + log2(len / 8), or 0 for the tile form.
__device__ int16_t wide_stage_form(const WideSlot &S, const double *longest, double *s_red)
{
    double m = 0.0;
    for (int32_t i = threadIdx.x; i < S.nvb; i += kWideThreads) m = fmax(m, longest[i]);
#pragma unroll
    for (int d = kWave / 2; d > 0; d /= 2) m = fmax(m, __shfl_xor(m, d));
    __syncthreads();
    if (lane_id() == 0) s_red[threadIdx.x / kWave] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWideWaves; ++w) m = fmax(m, s_red[w]);
    if (S.nnz < kStageMinNnz || S.nnz > INT32_MAX - kStageMinNnz) return 0;
    for (int f = 0; f < kWideStageForms; ++f) {
        const int64_t len = 8 << f;
        if (m <= (double)len) return 2 * S.nnz >= len * S.n ? (int16_t)(f + 1) : (int16_t)0;
    }
    return 0;
}

// Staged-rows form of one virtual tile (see csr_stage_kernel): rows
// [k * 512 >> sh, + 512 >> sh) with 1 << sh lanes per row, each wavefront two
// blocks of 64 >> sh rows, the second one copied into LDS while the first
// one's gathers are in flight. Tiles past the last row write zero partials.
// kVec: 16-byte copies; arrays that these cannot read are copied 4 bytes per
// lane, to the same places.
template <bool kVec>
__device__ __forceinline__ void wide_stage_tile(unsigned char *s_raw, double *s_red, int32_t k, const WideSlot &S,
                                                int sh, const double *src, double *y, const double *dw)
{
    constexpr int kCap = kWideStageCap, kLen = 8;
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double *s_val = reinterpret_cast<double *>(s_raw + (size_t)wid * kCap * (sizeof(double) + sizeof(int32_t)));
    int32_t *s_col = reinterpret_cast<int32_t *>(s_val + kCap);
    const int g = lane >> sh, sl = lane & ((1 << sh) - 1);
    const int32_t per = kWave >> sh;  // rows per block
    const int32_t n = S.n;
    const int32_t nnz8 = (int32_t)(S.nnz & ~(int64_t)7);
    const int32_t first = (k * kWideStageWaves + wid) * 2 * per;  // below 2^31: k < ntiles
    __syncthreads();  // LDS of a previous tile handled by this work-group is consumed
    double d1 = 0.0, d2 = 0.0;
    if (first < n) {
        int32_t ra[2], rb[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int32_t r = first + t * per + g;
            ra[t] = S.rowptr[r < n ? r : n];
            rb[t] = S.rowptr[r + 1 < n ? r + 1 : n];
        }
        double wv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int32_t r = first + t * per + g;
            wv[t] = sl == 0 && r < n ? dw[r] : 0.0;
        }
        auto stage = [&](int32_t s, int32_t e) {
            const int32_t a0 = s & ~3;
            const int32_t lim = e < nnz8 ? e : nnz8;
            const int32_t last = lim > 0 ? lim - 1 : 0;
            if constexpr (kVec) {
                const int32_t lastc = last & ~3, lastv = last & ~1;
#pragma unroll
                for (int u = 0; u < kCap / (4 * kWave); ++u) {
                    const int32_t p = a0 + (u * kWave + lane) * 4;
                    wide_copy<16>(S.col + (p < lastc ? p : lastc), s_col + u * kWave * 4);
                }
#pragma unroll
                for (int u = 0; u < kCap / (2 * kWave); ++u) {
                    const int32_t p = a0 + (u * kWave + lane) * 2;
                    wide_copy<16>(S.val + (p < lastv ? p : lastv), s_val + u * kWave * 2);
                }
            } else {
#pragma unroll 1
                for (int u = 0; u < kCap / kWave; ++u) {
                    const int32_t p = a0 + u * kWave + lane;
                    wide_copy<4>(S.col + (p < last ? p : last), s_col + u * kWave);
                }
                const int32_t *words = reinterpret_cast<const int32_t *>(S.val);  // two to a value
#pragma unroll 1
                for (int u = 0; u < 2 * kCap / kWave; ++u) {
                    const int64_t q = 2 * (int64_t)a0 + u * kWave + lane, most = 2 * (int64_t)last + 1;
                    wide_copy<4>(words + (q < most ? q : most), reinterpret_cast<int32_t *>(s_val) + u * kWave);
                }
            }
        };
        stage(__builtin_amdgcn_readfirstlane(ra[0]), readlane(rb[0], kWave - 1));
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies have landed
            const int32_t a0 = __builtin_amdgcn_readfirstlane(ra[t]) & ~3;
            const int32_t lim = nnz8 - a0 > kCap ? a0 + kCap : nnz8;  // staged: [a0, lim)
            const int32_t pe = rb[t] < lim ? rb[t] : lim;
            int32_t c[kLen];
            double v[kLen], xv[kLen];
#pragma unroll
            for (int u = 0; u < kLen; ++u) {
                const int32_t p = ra[t] + sl + (u << sh);
                const int32_t q = p < pe ? p - a0 : 0;
                c[u] = s_col[q];
                v[u] = s_val[q];
                if (p >= pe) c[u] = 0;
            }
#pragma unroll
            for (int u = 0; u < kLen; ++u) xv[u] = src[c[u]];
            if (t == 0) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this block's LDS reads are done
                stage(__builtin_amdgcn_readfirstlane(ra[1]), readlane(rb[1], kWave - 1));
            }
            double sum = 0.0;
#pragma unroll
            for (int u = 0; u < kLen; ++u) {
                const double f = sum + v[u] * xv[u];
                sum = ra[t] + sl + (u << sh) < pe ? f : sum;
            }
            // the row's entries past the stage
            for (int32_t p = ra[t] + sl; p < rb[t]; p += 1 << sh)
                if (p >= lim) sum += S.val[p] * src[S.col[p]];
            sum = subwave_sum_dyn(sum, 1 << sh);
            const int32_t r = first + t * per + g;
            if (sl == 0 && r < n) {
                y[r] = sum;
                d1 += sum * wv[t];
                d2 += sum * sum;
            }
        }
    }
    d1 = block_sum<double, kCsrThreads>(d1, s_red);
    d2 = block_sum<double, kCsrThreads>(d2, s_red);
    const double v[2] = {d1, d2};
    write_partials<double, 2>(v, S.part_a, S.ntiles, k);
}

// Product phase: one work-group per virtual tile (system, tile). Both forms
// run with their dot epilogue in both modes (w.r in the run mode; the
// true-residual mode multiplies x and ignores the partial).
// What bounds it: the matrix stream, out of the Infinity Cache once the
// systems' matrices and vectors fit there. Measured on one MI355X, 16 Poisson
// grids of 1.9 million rows together (143 MB per product): tile form 48 us,
// staged form 29.6 us (4.8 TB/s); non-temporal copies, which the single
// product uses, 39. Six work-groups per CU against five: 29.6 / 30.4 us.
// Runs of 4, 16 and 64 tiles per XCD: 29.4 / 30.4 / 32.8 us (at five). 17
// random columns per row (1.7 million rows) take the tile form: 185 us.
__global__ __launch_bounds__(kCsrThreads, 6) void wide_a_kernel(const WideSlot *__restrict__ slots,
                                                             const WideState *__restrict__ st,
                                                             const WideMap *__restrict__ map,
                                                             const int32_t *__restrict__ ta_slot,
                                                             const int32_t *__restrict__ ta_local)
{
    constexpr size_t kTileLds = csr_tile_lds<double, double, kCsrTile, kCsrLateGather>();
    constexpr size_t kStageLds = (size_t)kWideStageWaves * kWideStageCap * (sizeof(double) + sizeof(int32_t));
    __shared__ __align__(16) unsigned char s_raw[kTileLds > kStageLds ? kTileLds : kStageLds];
    __shared__ double s_red[kWideWaves];
    const int32_t total = map->total_ta;
    // XCD j takes runs of kWideRunTiles consecutive tiles: neighbouring rows share
    // its L2, and every XCD has its share of every large system
    constexpr int32_t kGroup = kWideRunTiles * kXcds;
    const int32_t padded = (total + kGroup - 1) / kGroup * kGroup;
    for (int32_t i = blockIdx.x; i < padded; i += gridDim.x) {
        const int32_t w = i % kGroup;
        const int32_t v = i - w + (w % kXcds) * kWideRunTiles + w / kXcds;
        if (v >= total) continue;
        const int32_t s = ta_slot[v], k = ta_local[v];
        const int32_t mode = st[s].mode;
        if (mode != kWideRun && mode != kWideCheck) continue;
        const WideSlot S = slots[s];
        // one instantiation of each form for every case; the second partial
        // (y.y) is used by BiCGSTAB's t = A s only
        const double *src = mode == kWideRun ? S.r : S.x;
        const double *dw = src;
        double *y = S.w;
        if (S.solver == kSlotBicgstab && mode == kWideRun) {
            const int32_t bp = st[s].bphase;
            if (bp == 0) {  // v = A p, r_hat.v
                src = S.p;
                dw = S.rh;
            } else if (bp == 1) {  // t = A s (s is held in r), t.s and t.t
                y = S.t;
            } else {
                continue;  // no product in this pair
            }
        }
        const int form = st[s].stage;
        if (form > 0 && ((reinterpret_cast<uintptr_t>(S.col) | reinterpret_cast<uintptr_t>(S.val)) & 15) == 0)
            wide_stage_tile<true>(s_raw, s_red, k, S, form - 1, src, y, dw);
        else if (form > 0)
            wide_stage_tile<false>(s_raw, s_red, k, S, form - 1, src, y, dw);
        else
            csr_tile<double, double, 2, kCsrThreads, kCsrTile, 1, kCsrLateGather>(
                s_raw, k, S.n, S.nnz, S.ntiles, S.rowptr, S.col, S.val, src, y, 1.0, 0.0, dw, S.part_a, S.csr_part);
    }
}

enum WideStep : int32_t { kStepTake = 0, kStepCheck = 1, kStepDone = 2 };

// The run mode's decision, taken alike by every block of the system from the
// two sums gamma = r.r and delta = r.w. On kStepTake, alpha and beta are set;
// on kStepDone, W holds the final status.
__device__ int32_t run_decision(WideState &W, const WideSlot &S, double gamma, double delta, double &alpha,
                                double &beta)
{
    W.spmv += 1;
    const double bb = W.truer == 2 ? gamma : W.bb;  // r = b: gamma is b.b
    W.bb = bb;
    W.rr = gamma;
    if (!__builtin_isfinite(gamma)) {
        W.status = kSlotNonfinite;
        return kStepDone;
    }
    if (gamma <= S.tol2 * bb) {  // also b = 0 (gamma = bb = 0)
        if (W.truer == 0) return kStepCheck;
        W.status = kSlotConverged;
        W.relres_true = bb > 0.0 ? sqrt(gamma / bb) : 0.0;
        return kStepDone;
    }
    if (W.iters >= S.maxit) {
        W.status = kSlotMaxit;
        return kStepDone;
    }
    beta = W.restart ? 0.0 : gamma / W.rho;
    const double den = W.restart ? delta : delta - beta * gamma / W.alpha;
    if (!__builtin_isfinite(delta) || !__builtin_isfinite(den)) {
        W.status = kSlotNonfinite;
        return kStepDone;
    }
    if (!(den > 0.0)) {  // p.A p <= 0: A is not positive definite along p
        W.status = kSlotBreakdown;
        return kStepDone;
    }
    alpha = gamma / den;
    return kStepTake;
}

// BiCGSTAB's vector phase on one virtual block of one system; the lead block
// commits the state to *next. part_in / part_out: two rows of nvb partials.
__device__ void bicgstab_vector_phase(const WideSlot &S, const WideState &W0, bool lead, int32_t lv,
                                      const double *part_in, double *part_out, WideState *next, double *s_red)
{
    const int32_t r0 = lv * kWideRows, r1 = min(S.n, r0 + kWideRows);
    WideState W = W0;
    int nw = 0;  // partial rows this block stores into part_out
    double t0 = 0.0, t1 = 0.0;
    auto done = [&](int32_t status) {
        W.status = status;
        W.mode = kWideDone;
        if (status != kSlotConverged) W.relres_true = W.bb > 0.0 ? sqrt(W.rr / W.bb) : 0.0;
    };
    if (W0.mode == kWideInit) {  // x = 0 (written at admission): r = r_hat = b
        for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) {
            const double bi = S.b[i];
            S.r[i] = bi;
            S.rh[i] = bi;
            t0 += bi * bi;
        }
        const double longest = wide_longest_row(S, r0, r1, s_red);
        if (threadIdx.x == 0) part_out[S.nvb + lv] = longest;
        nw = 1;
        W.mode = kWideRun;
        W.bphase = 3;
        W.truer = 2;
    } else if (W0.mode == kWideCheck) {  // r = b - A x (A x in w), r_hat = r
        for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) {
            const double ri = S.b[i] - S.w[i];
            S.r[i] = ri;
            S.rh[i] = ri;
            t0 += ri * ri;
        }
        nw = 1;
        W.spmv += 1;
        W.mode = kWideRun;
        W.bphase = 3;
        W.truer = 1;
    } else if (W0.bphase == 3) {  // a true residual's r.r: converged, or (re)start
        const double tr = wide_part_sum(part_in, S.nvb, s_red);
        if (W0.truer == 2) W.bb = tr;
        if (W0.truer == 2 && lead) W.stage = wide_stage_form(S, part_in + S.nvb, s_red);
        W.rr = tr;
        if (!__builtin_isfinite(tr)) {
            done(kSlotNonfinite);
        } else if (tr <= S.tol2 * W.bb) {  // also b = 0
            W.relres_true = W.bb > 0.0 ? sqrt(tr / W.bb) : 0.0;
            done(kSlotConverged);
        } else {
            for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) S.p[i] = S.r[i];
            W.rho = tr;  // r_hat = r
            W.rho0 = W.alpha = W.omega = 1.0;
            W.truer = 0;
            W.bphase = 0;
        }
    } else if (W0.bphase == 0) {  // v = A p is in w: alpha, s = r - alpha v
        const double rhv = wide_part_sum(S.part_a, S.ntiles, s_red);
        if (W0.iters >= S.maxit) {
            done(kSlotMaxit);
        } else {
            W.iters += 1;
            W.spmv += 1;
            if (!__builtin_isfinite(rhv)) {
                done(kSlotNonfinite);
            } else if (rhv == 0.0) {
                done(kSlotBreakdown);
            } else {
                const double alpha = W0.rho / rhv;
                for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) {
                    const double si = S.r[i] - alpha * S.w[i];
                    S.r[i] = si;
                    t0 += si * si;
                }
                nw = 1;
                W.alpha = alpha;
                W.bphase = 1;
            }
        }
    } else if (W0.bphase == 1) {  // t = A s is in t: omega, x, r = s - omega t
        const double ss = wide_part_sum(part_in, S.nvb, s_red);
        const double ts = wide_part_sum(S.part_a, S.ntiles, s_red);
        const double tt = wide_part_sum(S.part_a + S.ntiles, S.ntiles, s_red);
        W.rr = ss;
        const double alpha = W0.alpha;
        if (ss <= S.tol2 * W0.bb) {  // ||s|| small: x += alpha p, then confirm
            for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) S.x[i] += alpha * S.p[i];
            W.mode = kWideCheck;
        } else {
            W.spmv += 1;  // t = A s
            if (!__builtin_isfinite(tt) || !__builtin_isfinite(ss)) {
                done(kSlotNonfinite);
            } else if (tt == 0.0) {
                done(kSlotBreakdown);
            } else {
                const double omega = ts / tt;
                for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) {
                    const double si = S.r[i];
                    S.x[i] += alpha * S.p[i] + omega * si;
                    const double ri = si - omega * S.t[i];
                    S.r[i] = ri;
                    t0 += ri * ri;
                    t1 += S.rh[i] * ri;
                }
                nw = 2;
                W.omega = omega;
                W.bphase = 2;
            }
        }
    } else {  // bphase 2: r.r and r_hat.r: confirm, or beta and p
        const double rr = wide_part_sum(part_in, S.nvb, s_red);
        const double rho = wide_part_sum(part_in + S.nvb, S.nvb, s_red);
        W.rr = rr;
        if (!__builtin_isfinite(rr)) {
            done(kSlotNonfinite);
        } else if (rr <= S.tol2 * W0.bb) {
            W.mode = kWideCheck;
        } else if (W0.omega == 0.0 || rho == 0.0) {
            done(kSlotBreakdown);
        } else if (!__builtin_isfinite(rho)) {
            done(kSlotNonfinite);
        } else {
            const double beta = (rho / W0.rho) * (W0.alpha / W0.omega);
            const double omega = W0.omega;
            for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads)
                S.p[i] = S.r[i] + beta * (S.p[i] - omega * S.w[i]);
            W.rho0 = W0.rho;
            W.rho = rho;
            W.bphase = 0;
        }
    }
    if (nw > 0) {
        t0 = wide_wg_sum(t0, s_red);
        if (nw > 1) t1 = wide_wg_sum(t1, s_red);
        if (threadIdx.x == 0) {
            part_out[lv] = t0;
            if (nw > 1) part_out[S.nvb + lv] = t1;
        }
        W.phase = W0.phase ^ 1;
    }
    if (lead && threadIdx.x == 0) *next = W;
}

// Vector phase and commit; bound by its nine vector streams. The rows of a
// block are loaded before the sums that scale them are formed: 1.9 million
// rows 26.9 -> 24.3 us (5.7 TB/s). Every block reads this iteration's state
// from st; the first virtual block of each system writes the updated state
// to st_next (the two buffers alternate from one iteration to the next).
__global__ __launch_bounds__(kWideThreads, 6) void wide_v_kernel(const WideSlot *__restrict__ slots,
                                                              const WideState *__restrict__ st,
                                                              WideState *__restrict__ st_next,
                                                              const WideMap *__restrict__ map,
                                                              const int32_t *__restrict__ vb_slot,
                                                              const int32_t *__restrict__ vb_local)
{
    __shared__ double s_red[kWideWaves];
    const int32_t total = map->total_vb;
    for (int32_t v = blockIdx.x; v < total; v += gridDim.x) {
        const int32_t s = vb_slot[v], lv = vb_local[v];
        const WideState W0 = st[s];
        const bool lead = lv == 0;  // this block commits the system's state
        if (W0.mode == kWideDone) {
            if (lead && threadIdx.x == 0) st_next[s] = W0;
            continue;
        }
        const WideSlot S = slots[s];
        const int32_t r0 = lv * kWideRows, r1 = min(S.n, r0 + kWideRows);
        const double *part_in = S.part + (W0.phase ? 2 * S.nvb : 0);
        double *part_out = S.part + (W0.phase ? 0 : 2 * S.nvb);
        if (S.solver == kSlotBicgstab) {
            bicgstab_vector_phase(S, W0, lead, lv, part_in, part_out, st_next + s, s_red);
            continue;
        }
        WideState W = W0;
        bool wrote = false;  // this block stored a partial into part_out
        double t = 0.0;
        if (W0.mode == kWideRun) {
            // the block's vectors do not wait for the sums that scale them
            constexpr int kPer = kWideRows / kWideThreads;
            double rv[kPer], wv[kPer], pv[kPer], sv[kPer], xv[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int32_t i = r0 + u * kWideThreads + threadIdx.x;
                rv[u] = wv[u] = pv[u] = sv[u] = xv[u] = 0.0;
                if (i < r1) {
                    rv[u] = S.r[i];
                    wv[u] = S.w[i];
                    xv[u] = S.x[i];
                    if (!W0.restart) {
                        pv[u] = S.p[i];
                        sv[u] = S.s[i];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            const double gamma = wide_part_sum(part_in, S.nvb, s_red);
            const double delta = wide_part_sum(S.part_a, S.ntiles, s_red);
            if (W0.truer == 2 && lead) W.stage = wide_stage_form(S, part_in + S.nvb, s_red);
            double alpha = 0.0, beta = 0.0;
            const int32_t step = run_decision(W, S, gamma, delta, alpha, beta);
            if (step == kStepTake) {
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int32_t i = r0 + u * kWideThreads + threadIdx.x;
                    if (i < r1) {
                        const double pi = W0.restart ? rv[u] : rv[u] + beta * pv[u];
                        const double si = W0.restart ? wv[u] : wv[u] + beta * sv[u];
                        S.p[i] = pi;
                        S.s[i] = si;
                        S.x[i] = xv[u] + alpha * pi;
                        const double ri = rv[u] - alpha * si;
                        S.r[i] = ri;
                        t += ri * ri;
                    }
                }
                wrote = true;
                W.iters += 1;
                W.rho = gamma;
                W.alpha = alpha;
                W.restart = 0;
                W.truer = 0;
            } else if (step == kStepCheck) {
                W.mode = kWideCheck;
            } else {
                W.mode = kWideDone;
                if (W.status != kSlotConverged) W.relres_true = W.bb > 0.0 ? sqrt(W.rr / W.bb) : 0.0;
            }
        } else if (W0.mode == kWideCheck) {
            for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) {
                const double ri = S.b[i] - S.w[i];
                S.r[i] = ri;
                t += ri * ri;
            }
            wrote = true;
            W.spmv += 1;
            W.mode = kWideRun;
            W.restart = 1;
            W.truer = 1;
        } else {  // init: x = 0 was written at admission
            for (int32_t i = r0 + threadIdx.x; i < r1; i += kWideThreads) {
                const double bi = S.b[i];
                S.r[i] = bi;
                t += bi * bi;
            }
            const double longest = wide_longest_row(S, r0, r1, s_red);
            if (threadIdx.x == 0) part_out[S.nvb + lv] = longest;
            wrote = true;
            W.mode = kWideRun;
            W.restart = 1;
            W.truer = 2;
        }
        if (wrote) {
            t = wide_wg_sum(t, s_red);
            if (threadIdx.x == 0) part_out[lv] = t;
            W.phase = W0.phase ^ 1;
        }
        if (lead && threadIdx.x == 0) st_next[s] = W;
    }
}

spx_status wide_iteration_launch(const WideSlot *slots, const WideState *st, WideState *st_next,
                                 const WideMap *map, const int32_t *vb_slot, const int32_t *vb_local,
                                 const int32_t *ta_slot, const int32_t *ta_local, int grid, hipStream_t stream)
{
    wide_a_kernel<<<grid, kCsrThreads, 0, stream>>>(slots, st, map, ta_slot, ta_local);
    SPX_LAUNCHED();
    wide_v_kernel<<<grid, kWideThreads, 0, stream>>>(slots, st, st_next, map, vb_slot, vb_local);
    SPX_LAUNCHED();
    return SPX_OK;
}

}  // namespace spx
