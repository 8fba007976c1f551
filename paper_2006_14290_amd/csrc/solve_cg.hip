// solve_cg.hip -- preconditioned conjugate gradients on the GPU.
//
// Textbook PCG (Hestenes & Stiefel 1952; the preconditioned form of Barrett
// et al., "Templates", 1994) with a scalar Jacobi preconditioner, the solver
// the paper benchmarks in Section 4. One iteration is three launches:
//   1. q = A p fused with the partial sums of p.q (CSR, ELL and SELL-P
//      epilogue; a separate dot kernel for the other formats);
//   2. alpha = rho / p.q, r -= alpha q, partial sums of r.r and r.z
//      (z = D^{-1} r is not stored; block Jacobi forms it in one more launch);
//   3. x += alpha p, beta and the test ||r|| <= tol ||b||, p = z + beta p.
// Every work-group of 2 and 3 sums the partials of the launch before it in
// the same fixed order. Where the product leaves more than 4,096 of them (tile
// kernel above 8.4 million entries, ELL above 1 or 2 million rows, SELL-P above
// 1 million, the separate dot kernel above 4.2 million rows), one work-group
// first sums them in a launch more (4.7 us).
// Scalars never leave the device; a block of `check_every` iterations is
// captured once into a hipGraph and replayed, and the host reads the state
// only between replays. When the recursive residual passes, the true residual
// b - A x decides; a miss restarts the recurrences from it.
// Small float64 CSR systems (at most kSmallMaxRows rows, scalar Jacobi or no
// preconditioner) run the whole solve in one launch instead (small_cg.hip).
// Float64 throughout for spx_cg_solve; the same driver runs in float32
// (float32 or binary16-stored matrix values) as the inner solver of
// mixed-precision iterative refinement.
#include <type_traits>

#include "convert.hpp"
#include "small_cg.hpp"
#include "solver_common.hpp"
#include "solvers.hpp"
#include "vec_io.hpp"

namespace spx {

// The fields of the state that an iteration reads, into another buffer.
__device__ __forceinline__ void cg_commit(const KState *in, KState *out, double rho, double rr, int32_t flag,
                                          int32_t iters, int32_t spmv_count)
{
    out->rho = rho;
    out->rr = rr;
    out->bb = in->bb;
    out->tol2 = in->tol2;
    out->maxit = in->maxit;
    out->flag = flag;
    out->iters = iters;
    out->spmv_count = spmv_count;
}

template <typename X>
__global__ __launch_bounds__(kVecThreads) void cg_init_kernel(int64_t n, const X *__restrict__ b,
                                                             const X *__restrict__ q, const X *__restrict__ dinv,
                                                             X *__restrict__ r, X *__restrict__ p,
                                                             X *__restrict__ partials, KState *st)
{
    __shared__ X s_red[kVecThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kVecChunk;
    X bb = X(0), rz = X(0), rr = X(0);
#pragma unroll
    for (int u = 0; u < kVecItems; ++u) {
        const int64_t i = base + threadIdx.x + u * kVecThreads;
        if (i < n) {
            const X bi = b[i];
            const X ri = q ? bi - q[i] : bi;
            const X zi = dinv ? ri * dinv[i] : ri;
            r[i] = ri;
            p[i] = zi;
            bb += bi * bi;
            rz += ri * zi;
            rr += ri * ri;
        }
    }
    X v[3] = {block_sum<X, kVecThreads>(bb, s_red), block_sum<X, kVecThreads>(rz, s_red),
              block_sum<X, kVecThreads>(rr, s_red)};
    write_partials<X, 3>(v, partials, gridDim.x, blockIdx.x);
}

// One iteration's two vector kernels. Both first sum the partials that the
// kernel before them left (every work-group the same ones in the same order,
// so all take the same decisions) instead of waiting for a one-work-group
// finisher in between; the loads of their first vectors are in flight
// meanwhile. At most kCgBlocks work-groups, so that the partials stay few
// (1,024 values: 8 KB per work-group and row, from L2). The product's are at
// most kMaxParts; block Jacobi's r.z, one per 1,024 rows, are summed as they
// are (first summed to one: 256^3, 16,384 of them, 716 us per iteration against
// 719, 164^3 178.6 against 177.4). What bounds the kernels: the
// vectors. Against the five-launch iteration (product, finisher, update,
// finisher, direction), on one MI355X: Jacobi on the anisotropic 128^3 grid 82
// -> 73 us per iteration (z is not stored: one vector pass less), the 64^3
// 7-point grid 25 -> 20, the 257^2 grid 14 -> 10.5.
constexpr int kCgBlocks = 1024;

inline int64_t cg_blocks(int64_t n)
{
    const int64_t b = vec_blocks(n);
    return b < kCgBlocks ? b : kCgBlocks;
}

// How z = M^{-1} r comes about: z = r, z = r * dinv, or z a vector of its own
// (block Jacobi).
enum CgPre : int { kCgNone = 0, kCgJacobi = 1, kCgBlock = 2 };

// alpha = rho / p.q; r -= alpha q; partials of r.r (and of r.z for kCgJacobi).
// The first work-group records alpha, or why there is none, for the second
// kernel (no work-group of this launch reads those two fields).
template <typename X, CgPre kPre>
__global__ __launch_bounds__(kVecThreads) void cg_residual_kernel(int64_t n, const X *__restrict__ pq, int npq,
                                                                 const X *__restrict__ q, X *__restrict__ r,
                                                                 const X *__restrict__ dinv, X *__restrict__ rr_out,
                                                                 X *__restrict__ rz_out, KState *st)
{
    if (st->flag != kRunning) return;
    __shared__ X s_red[kVecThreads / kWave];
    __shared__ double s_sum[kVecThreads / kWave];
    const int64_t step = (int64_t)gridDim.x * kVecChunk;
    int64_t i0 = vec_i0();
    vec4_t<X> rv = ld4<X, true>(r, i0, n), qv = ld4<X, true>(q, i0, n), dv = {};
    if (kPre == kCgJacobi) dv = ld4<X, true>(dinv, i0, n);
    const double t = block_sum_partials<X, kVecThreads>(pq, npq, s_sum);
    const int32_t stop = !finite(t) ? kNonfinite : (t <= 0.0 ? kBreakdown : kRunning);
    const double alpha = st->rho / t;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->pad0 = stop;
        st->alpha = alpha;
    }
    if (stop != kRunning) return;
    const X a = (X)alpha;
    X rz = X(0), rr = X(0);
    while (true) {
#pragma unroll
        for (int u = 0; u < kVecItems; ++u) {
            rv[u] = rv[u] - a * qv[u];
            if (kPre == kCgJacobi) rz += rv[u] * (rv[u] * dv[u]);
            rr += rv[u] * rv[u];
        }
        st4<X, true>(r, i0, n, rv);
        i0 += step;
        if (i0 - threadIdx.x * kVecItems >= n) break;  // uniform across the work-group
        rv = ld4<X, true>(r, i0, n);
        qv = ld4<X, true>(q, i0, n);
        if (kPre == kCgJacobi) dv = ld4<X, true>(dinv, i0, n);
    }
    X v[1] = {block_sum<X, kVecThreads>(rr, s_red)};
    write_partials<X, 1>(v, rr_out, gridDim.x, blockIdx.x);
    if (kPre == kCgJacobi) {
        v[0] = block_sum<X, kVecThreads>(rz, s_red);
        write_partials<X, 1>(v, rz_out, gridDim.x, blockIdx.x);
    }
}

// x += alpha p; beta = r.z / rho and the convergence test; p = z + beta p.
// The state after the iteration goes to another buffer than the one that this
// launch's work-groups read.
template <typename X, CgPre kPre, bool kVecX>
__global__ __launch_bounds__(kVecThreads) void cg_direction_kernel(int64_t n, const X *__restrict__ rr_in, int nrr,
                                                                  const X *__restrict__ rz_in, int nrz,
                                                                  const X *__restrict__ z, const X *__restrict__ dinv,
                                                                  X *__restrict__ x, X *__restrict__ p,
                                                                  const KState *__restrict__ in,
                                                                  KState *__restrict__ out)
{
    __shared__ double s_sum[kVecThreads / kWave];
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    int32_t flag = in->flag;
    if (flag == kRunning) flag = in->pad0;
    if (flag != kRunning) {
        if (first) cg_commit(in, out, in->rho, in->rr, flag, in->iters, in->spmv_count);
        return;
    }
    const int64_t step = (int64_t)gridDim.x * kVecChunk;
    int64_t i0 = vec_i0();
    vec4_t<X> xv = ld4<X, kVecX>(x, i0, n), pv = ld4<X, true>(p, i0, n), zv = ld4<X, true>(z, i0, n), dv = {};
    if (kPre == kCgJacobi) dv = ld4<X, true>(dinv, i0, n);
    const double rr = block_sum_partials<X, kVecThreads>(rr_in, nrr, s_sum);
    const double rz = kPre == kCgNone ? rr : block_sum_partials<X, kVecThreads>(rz_in, nrz, s_sum);
    const int32_t iters = in->iters + 1;
    if (!finite(rr) || !finite(rz)) flag = kNonfinite;
    else if (rr <= in->tol2 * in->bb) flag = kConverged;
    else if (iters >= in->maxit) flag = kMaxit;
    if (first) cg_commit(in, out, flag == kRunning || flag == kMaxit ? rz : in->rho, rr, flag, iters,
                         in->spmv_count + 1);
    const X a = (X)in->alpha, be = (X)(rz / in->rho);
    while (true) {
#pragma unroll
        for (int u = 0; u < kVecItems; ++u) {
            xv[u] += a * pv[u];
            pv[u] = (kPre == kCgJacobi ? zv[u] * dv[u] : zv[u]) + be * pv[u];
        }
        st4<X, kVecX>(x, i0, n, xv);
        if (flag == kRunning) st4<X, true>(p, i0, n, pv);
        i0 += step;
        if (i0 - threadIdx.x * kVecItems >= n) break;
        xv = ld4<X, kVecX>(x, i0, n);
        pv = ld4<X, true>(p, i0, n);
        zv = ld4<X, true>(z, i0, n);
        if (kPre == kCgJacobi) dv = ld4<X, true>(dinv, i0, n);
    }
}

// After an odd number of iterations: the state back to the first buffer.
__global__ void cg_state_copy_kernel(const KState *__restrict__ in, KState *__restrict__ out)
{
    if (threadIdx.x == 0) cg_commit(in, out, in->rho, in->rr, in->flag, in->iters, in->spmv_count);
}

template <typename X>
__global__ __launch_bounds__(kVecThreads) void cg_restart_kernel(int64_t n, const X *__restrict__ r,
                                                                const X *__restrict__ dinv, X *__restrict__ p,
                                                                X *__restrict__ partials, KState *st)
{
    __shared__ X s_red[kVecThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kVecChunk;
    X rz = X(0);
#pragma unroll
    for (int u = 0; u < kVecItems; ++u) {
        const int64_t i = base + threadIdx.x + u * kVecThreads;
        if (i < n) {
            const X ri = r[i];
            const X zi = dinv ? ri * dinv[i] : ri;
            p[i] = zi;
            rz += ri * zi;
        }
    }
    X v[1] = {block_sum<X, kVecThreads>(rz, s_red)};
    write_partials<X, 1>(v, partials, gridDim.x, blockIdx.x);
}

template <typename X>
__global__ void zero_kernel(int64_t n, X *__restrict__ x)
{
    const int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x;
    if (i < n) x[i] = X(0);
}

template <typename V, typename X>
struct CgBufs {
    X *r, *z, *p, *q, *d, *dinv, *partials;  // z: block Jacobi only, else r
    double *inv;  // block-Jacobi inverse blocks
    KState *st;
    int32_t *part;
};

template <typename V, typename X>
static CgBufs<V, X> cg_carve(Carve &c, const spx_matrix &A, int precond)
{
    const int64_t n = A.nrows;
    CgBufs<V, X> w{};
    w.st = c.take<KState>(2);
    w.r = c.take<X>(n);
    w.p = c.take<X>(n);
    w.q = c.take<X>(n);
    w.z = precond >= 2 ? c.take<X>(n) : w.r;
    w.d = precond == 1 ? c.take<X>(n) : nullptr;
    w.dinv = precond == 1 ? c.take<X>(n) : nullptr;
    w.inv = precond >= 2 ? c.take<double>(ceil_div(n, precond) * precond * precond) : nullptr;
    w.partials = c.take<X>(3 * partial_slots(A));
    w.part = (A.fmt == SPX_CSR && A.csr_part == nullptr) ? c.take<int32_t>(csr_partition_bytes(A.nnz) / 4) : nullptr;
    return w;
}

template <typename V, typename X>
size_t cg_workspace(const spx_matrix &A, int precond)
{
    Carve c(nullptr, 0);
    (void)cg_carve<V, X>(c, A, precond);
    return c.off + 256;
}

// The one-launch solve of a small float64 CSR system (small_cg.hip) and the
// same bookkeeping as the general driver.
static spx_status small_cg_finish(const spx_matrix &A, const double *b, double *x, const SolveSpec &sp,
                                  const CgBufs<double, double> &w, SolveEnv *env, spx_solve_info *info,
                                  hipStream_t user_stream)
{
    hipStream_t s = env->stream;
    const int64_t n = A.nrows;
    const bool cached = A.max_row_len > 0 && A.max_row_len <= kSmallCachedLen;
    SPX_CHECK(small_cg_launch(A, b, x, sp.precond ? w.dinv : nullptr, sp.x0_zero, cached, w.st, s));
    KState hs;
    SPX_CHECK(read_state(env, w.st, &hs));
    if (hs.flag == kLongRow) {  // the row-length hint was too small
        SPX_CHECK(state_set_flag(w.st, kRunning, s));
        SPX_CHECK(small_cg_launch(A, b, x, sp.precond ? w.dinv : nullptr, sp.x0_zero, false, w.st, s));
        SPX_CHECK(read_state(env, w.st, &hs));
    }
    double true2 = hs.tmp[0];
    if (true2 < 0.0 && hs.bb > 0.0) {  // stopped before a true residual was formed
        SPX_CHECK(spmv_dispatch(A, x, w.q, 1.0, 0.0, s));
        SPX_CHECK(residual_norm<double>(n, b, w.q, w.r, w.partials, w.st, s));
        KState h2;
        SPX_CHECK(read_state(env, w.st, &h2));
        true2 = h2.tmp[0];
    }
    spx_status status = status_of_flag(hs.flag);
    if (hs.flag == kMaxit) set_error("cg: no convergence in %d iterations", sp.maxit);
    else if (hs.flag == kBreakdown) set_error("cg: breakdown (p'Ap <= 0)");
    else if (hs.flag == kNonfinite) set_error("cg: non-finite residual");
    SPX_HIP(hipEventRecord(env->ev1, s));
    SPX_HIP(hipEventSynchronize(env->ev1));
    float ms = 0.f;
    SPX_HIP(hipEventElapsedTime(&ms, env->ev0, env->ev1));
    info->status = status;
    info->iters = hs.iters;
    info->spmv_count = hs.spmv_count;
    info->relres_recursive = hs.bb > 0 ? sqrt(hs.rr / hs.bb) : 0.0;
    info->relres_true = hs.bb > 0 ? sqrt(true2 / hs.bb) : 0.0;
    info->device_ms = ms;
    SPX_HIP(hipEventRecord(env->join, s));
    SPX_HIP(hipStreamWaitEvent(user_stream, env->join, 0));
    return status;
}

template <typename V, typename X>
spx_status cg_run(const spx_matrix &A_in, const X *b, X *x, const SolveSpec &sp, void *ws, size_t ws_bytes,
                  spx_solve_info *info, hipStream_t user_stream)
{
    SolveEnv *env = nullptr;
    SPX_CHECK(solve_env(&env));
    hipStream_t s = env->stream;
    const int64_t n = A_in.nrows;
    Carve c(ws, ws_bytes);
    CgBufs<V, X> w = cg_carve<V, X>(c, A_in, sp.precond);
    SPX_REQUIRE(c.fits(), SPX_ERR_ARG, "cg: workspace of %zu bytes is too small (need %zu)", ws_bytes,
                cg_workspace<V, X>(A_in, sp.precond));
    spx_matrix A = A_in;
    *info = spx_solve_info{};

    SPX_HIP(hipEventRecord(env->join, user_stream));
    SPX_HIP(hipStreamWaitEvent(s, env->join, 0));
    SPX_HIP(hipEventRecord(env->ev0, s));
    // small float64 CSR systems: the whole solve in one work-group, one launch
    const bool small = std::is_same<V, double>::value && std::is_same<X, double>::value && A.fmt == SPX_CSR &&
                       n <= kSmallMaxRows && sp.precond <= 1 && sp.confirm_true;
    if (w.part && !small) {
        SPX_CHECK(csr_partition_launch(A, w.part, s));
        A.csr_part = w.part;
    }
    SPX_CHECK(state_init(w.st, sp.tol, sp.maxit, s));
    KState hs;
    const int32_t bs = sp.precond >= 2 ? sp.precond : 0;  // block-Jacobi block size
    if (sp.precond) {
        if (bs) SPX_CHECK(bj_setup<V>(A, bs, w.inv, w.st, s));
        else SPX_CHECK((jacobi_setup<V, X>(A, w.d, w.dinv, w.st, s)));
        SPX_CHECK(read_state(env, w.st, &hs));
        if (hs.flag != kRunning) {
            set_error(bs ? "cg: singular or non-finite diagonal block" : "cg: zero, missing or non-finite diagonal entry");
            return SPX_ERR_ZERO_DIAG;
        }
    }
    if constexpr (std::is_same<V, double>::value && std::is_same<X, double>::value) {
        if (small) return small_cg_finish(A, b, x, sp, w, env, info, user_stream);
    }
    const unsigned gv = (unsigned)vec_blocks(n);
    if (sp.x0_zero) {
        zero_kernel<X><<<(unsigned)ceil_div(n, kVecThreads), kVecThreads, 0, s>>>(n, x);
        cg_init_kernel<X><<<gv, kVecThreads, 0, s>>>(n, b, nullptr, w.dinv, w.r, w.p, w.partials, w.st);
    } else {
        SPX_CHECK(spmv_dispatch(A, x, w.q, 1.0, 0.0, s));
        cg_init_kernel<X><<<gv, kVecThreads, 0, s>>>(n, b, w.q, w.dinv, w.r, w.p, w.partials, w.st);
    }
    SPX_LAUNCHED();
    // block Jacobi: z = M^{-1} r, p = z and the r.z partials (row 1 of the init sums)
    if (bs) SPX_CHECK(bj_apply<X>(n, bs, w.inv, w.r, w.z, w.p, w.partials, 1, w.st, false, s));
    SPX_CHECK(launch_finish<X>(w.partials, gv, 3, w.st, kOpCgInit, s));
    SPX_CHECK(read_state(env, w.st, &hs));

    GraphGuard graph;
    const int m = sp.check_every > 0 ? sp.check_every : 16;
    // vector loads need every vector aligned to kVecItems entries (x is the
    // caller's; the workspace pieces are 256-byte aligned)
    const bool vec = (reinterpret_cast<uintptr_t>(x) % (kVecItems * sizeof(X))) == 0;
    const int64_t slots = partial_slots(A);
    X *rr_parts = w.partials + slots, *rz_parts = w.partials + 2 * slots;
    const unsigned gc = (unsigned)cg_blocks(n);
    const int nrz = bs ? (int)gv : (int)gc;
#define SPX_CG_RESIDUAL(PRE)                                                                                   \
    cg_residual_kernel<X, PRE><<<gc, kVecThreads, 0, s>>>(n, w.partials, (int)npq, w.q, w.r, w.dinv, rr_parts, \
                                                          rz_parts, in)
#define SPX_CG_DIRECTION(PRE, VEC)                                                                                   \
    cg_direction_kernel<X, PRE, VEC><<<gc, kVecThreads, 0, s>>>(n, rr_parts, (int)gc, rz_parts, nrz, bs ? w.z : w.r, \
                                                                w.dinv, x, w.p, in, out)
    auto iterations = [&]() -> spx_status {
        KState *in = w.st, *out = w.st + 1;
        for (int it = 0; it < m; ++it) {
            int64_t npq = 0;
            SPX_CHECK((spmv_dot_partials<V, X>(A, w.p, w.q, w.p, w.partials, in, &npq, s)));
            if (sp.precond == 1) SPX_CG_RESIDUAL(kCgJacobi);
            else SPX_CG_RESIDUAL(kCgNone);
            // block Jacobi: z = M^{-1} r and the r.z partials
            if (bs) SPX_CHECK(bj_apply<X>(n, bs, w.inv, w.r, w.z, nullptr, rz_parts, 0, in, true, s));
            if (bs) {
                if (vec) SPX_CG_DIRECTION(kCgBlock, true);
                else SPX_CG_DIRECTION(kCgBlock, false);
            } else if (sp.precond == 1) {
                if (vec) SPX_CG_DIRECTION(kCgJacobi, true);
                else SPX_CG_DIRECTION(kCgJacobi, false);
            } else {
                if (vec) SPX_CG_DIRECTION(kCgNone, true);
                else SPX_CG_DIRECTION(kCgNone, false);
            }
            SPX_LAUNCHED();
            KState *t = in;
            in = out;
            out = t;
        }
        if (m % 2) {
            cg_state_copy_kernel<<<1, kWave, 0, s>>>(in, out);
            SPX_LAUNCHED();
        }
        return SPX_OK;
    };
#undef SPX_CG_RESIDUAL
#undef SPX_CG_DIRECTION
    spx_status status = SPX_OK;
    bool have_true = false;
    double true2 = 0.0;
    while (true) {
        if (hs.flag == kZeroRhs) {
            zero_kernel<X><<<(unsigned)ceil_div(n, kVecThreads), kVecThreads, 0, s>>>(n, x);
            SPX_LAUNCHED();
            status = SPX_OK;
            have_true = true;
            true2 = 0.0;
            break;
        }
        if (hs.flag == kConverged) {
            if (!sp.confirm_true) {
                status = SPX_OK;
                break;
            }
            SPX_CHECK(spmv_dispatch(A, x, w.q, 1.0, 0.0, s));
            SPX_CHECK(residual_norm<X>(n, b, w.q, w.r, w.partials, w.st, s));
            SPX_CHECK(read_state(env, w.st, &hs));
            have_true = true;
            true2 = hs.tmp[0];
            if (true2 <= hs.tol2 * hs.bb) {
                status = SPX_OK;
                break;
            }
            if (hs.iters >= sp.maxit) {
                status = SPX_ERR_NOT_CONVERGED;
                break;
            }
            // restart the recurrences from the true residual (already in r)
            cg_restart_kernel<X><<<gv, kVecThreads, 0, s>>>(n, w.r, w.dinv, w.p, w.partials, w.st);
            SPX_LAUNCHED();
            if (bs) SPX_CHECK(bj_apply<X>(n, bs, w.inv, w.r, w.z, w.p, w.partials, 0, w.st, false, s));
            SPX_CHECK(launch_finish<X>(w.partials, gv, 1, w.st, kOpCgRestart, s));
            SPX_CHECK(read_state(env, w.st, &hs));
            have_true = false;
            continue;
        }
        if (hs.flag != kRunning) {
            status = status_of_flag(hs.flag);
            if (hs.flag == kMaxit) set_error("cg: no convergence in %d iterations", sp.maxit);
            else if (hs.flag == kBreakdown) set_error("cg: breakdown (p'Ap <= 0)");
            else set_error("cg: non-finite residual");
            break;
        }
        if (graph.exec == nullptr) SPX_CHECK(capture_graph(s, &graph.exec, iterations));
        SPX_HIP(hipGraphLaunch(graph.exec, s));
        SPX_CHECK(read_state(env, w.st, &hs));
    }
    if (!have_true && hs.bb > 0.0) {
        SPX_CHECK(spmv_dispatch(A, x, w.q, 1.0, 0.0, s));
        SPX_CHECK(residual_norm<X>(n, b, w.q, w.r, w.partials, w.st, s));
        KState h2;
        SPX_CHECK(read_state(env, w.st, &h2));
        true2 = h2.tmp[0];
    }
    SPX_HIP(hipEventRecord(env->ev1, s));
    SPX_HIP(hipEventSynchronize(env->ev1));
    float ms = 0.f;
    SPX_HIP(hipEventElapsedTime(&ms, env->ev0, env->ev1));
    info->status = status;
    info->iters = hs.iters;
    info->spmv_count = hs.spmv_count + (sp.x0_zero ? 0 : 1);
    info->relres_recursive = hs.bb > 0 ? sqrt(hs.rr / hs.bb) : 0.0;
    info->relres_true = hs.bb > 0 ? sqrt(true2 / hs.bb) : 0.0;
    info->device_ms = ms;
    SPX_HIP(hipEventRecord(env->join, s));
    SPX_HIP(hipStreamWaitEvent(user_stream, env->join, 0));
    return status;
}

template size_t cg_workspace<double, double>(const spx_matrix &, int);
template size_t cg_workspace<float, float>(const spx_matrix &, int);
template size_t cg_workspace<_Float16, float>(const spx_matrix &, int);
template spx_status cg_run<double, double>(const spx_matrix &, const double *, double *, const SolveSpec &, void *,
                                           size_t, spx_solve_info *, hipStream_t);
template spx_status cg_run<float, float>(const spx_matrix &, const float *, float *, const SolveSpec &, void *,
                                         size_t, spx_solve_info *, hipStream_t);
template spx_status cg_run<_Float16, float>(const spx_matrix &, const float *, float *, const SolveSpec &, void *,
                                            size_t, spx_solve_info *, hipStream_t);

}  // namespace spx
