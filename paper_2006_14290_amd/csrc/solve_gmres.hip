// solve_gmres.hip -- restarted, right-preconditioned GMRES(m) on the GPU.
//
// GMRES (Saad & Schultz 1986) as listed among the paper's solvers
// (Section 1), right-preconditioned with the scalar Jacobi M = diag(A):
// the Krylov space is that of A M^{-1}, and x = x0 + M^{-1} V y.
// Arnoldi orthogonalisation is classical Gram-Schmidt applied twice (CGS2,
// "twice is enough": Giraud, Langou, Rozloznik 2005) in three passes over the
// basis instead of four: h = V^T w; then w' = w - V h and V^T w' in one pass
// (a thread keeps its row of the basis in registers between the two); then
// w'' = w' - V h2 with ||w''||^2. The basis is stored unscaled: column k holds
// u_k = v_k / s_k, scaled to about unit length before its norm is known (by
// ||w'||, the norm before the second pass), with the exact 1 / ||u_k|| kept as
// the scalar s_k; products, dots and updates apply the scalars, so no kernel
// normalises. The last pass also writes z = M^{-1} u for the next product.
//
// Layout: rows in panels of 256, a panel's basis columns one after another
// (column k of panel p at (p (m + 1) + k) 256), so that a pass reads one
// contiguous stretch per panel instead of one short piece of each of up to
// m + 1 arrays n values apart.
// One-work-group-per-row finishers sum the partials; the step finisher builds
// the Hessenberg column, applies the previous Givens rotations, forms the new
// one, updates the residual estimate |g_{j+1}| and decides whether the cycle
// ends (estimate below tolerance, lucky breakdown, or maxit). All of this
// stays on the device; one restart cycle (m Arnoldi steps) is a single
// captured hipGraph, replayed per cycle. At the end of a cycle one wavefront
// stages the triangle of H and g in LDS and one of its lanes back-substitutes
// H y = g there; then x += M^{-1} V y, and the next cycle starts from the true
// residual b - A x.
//
// What bounds a step: the basis, (j + 1) n values per pass, read at 5.6 to 6
// TB/s.
// GMRES(30) + Jacobi, convection-diffusion 128^3, one MI355X: 283 us per step
// with four passes, 100 barriers per work-group and a normalising kernel,
// 202 us now.
#include <cmath>

#include "solver_common.hpp"
#include "solvers.hpp"

namespace spx {

using X = double;

struct GmState {
    int m;
    double *H;   // (m+1) x m, column-major: H[j*(m+1) + i]
    double *g;   // m+1
    double *cs;  // m
    double *sn;  // m
    double *y;   // m
    double *s;   // m+1: v_k = s_k u_k
    double *h1;  // m: first and second orthogonalisation coefficients
    double *h2;  // m
};

constexpr int kGmThreads = 256;  // = rows per panel
constexpr int kGmGroup = 4;      // basis vectors per unrolled group
constexpr int kGmBlocks = 2048;  // work-groups of a pass at most

static int64_t gm_panels(int64_t n) { return n > 0 ? ceil_div(n, kGmThreads) : 1; }

// Work-groups of a pass over nv basis vectors: as many per CU as stay resident
// with the registers that a thread's row of the basis and its sums take (32
// vectors: 164).
constexpr int gm_resident(int groups, bool update)
{
    return update ? (groups <= 2 ? 8 : (groups <= 4 ? 5 : (groups <= 6 ? 4 : (groups <= 8 ? 3 : (groups <= 13 ? 2 : 1)))))
                  : (groups <= 3 ? 8 : (groups <= 5 ? 5 : (groups <= 7 ? 4 : (groups <= 9 ? 3 : (groups <= 15 ? 2 : 1)))));
}

static int64_t gm_blocks(int64_t n, int nv, bool update)
{
    const int64_t most = 256 * gm_resident((nv + kGmGroup - 1) / kGmGroup, update);
    const int64_t b = gm_panels(n);
    return b < most ? b : most;
}

// Whether nv basis vectors are read as a stream (non-temporal) or left in the
// Infinity Cache (256 MB) for the next pass. 128^3, us a pass, plain /
// non-temporal: 12 vectors (201 MB) 28 / 37, 16: 38 / 48, 20: 55 / 59, 24 (403
// MB): 70 / 67, 28: 79 / 77; with the update 24: 74 / 69, 28: 88 / 78.
static int gm_streams(int64_t n, int nv) { return (int64_t)nv * n * (int64_t)sizeof(X) > (int64_t)360 << 20; }

// cycle start: u_0 = r / ||r|| (r in z, ||r||^2 in st->tmp[0]), z = M^{-1} u_0, g = ||r|| e1
__global__ __launch_bounds__(kGmThreads) void gm_cycle_init_kernel(int64_t n, const X *__restrict__ dinv,
                                                                  X *__restrict__ V, X *__restrict__ z, KState *st,
                                                                  GmState gs)
{
    const double beta = sqrt(st->tmp[0]);
    const int64_t i = (int64_t)blockIdx.x * kGmThreads + threadIdx.x;
    if (i < n) {
        const X v = z[i] / beta;
        V[(int64_t)blockIdx.x * (gs.m + 1) * kGmThreads + threadIdx.x] = v;
        z[i] = dinv ? v * dinv[i] : v;
    }
    if (i == 0) {
        for (int k = 0; k <= gs.m; ++k) gs.g[k] = 0.0;
        gs.g[0] = beta;
        gs.s[0] = 1.0;
        st->jend = 0;
        st->flag = kRunning;
    }
}

// One pass over the basis, thread per row. kUpdate: w = scale * w - sum_k
// dots[k] u_k first (scale = s_{nv-1}: w is the product with the unscaled
// u_{nv-1}); then, always, the partials of u_k . w at partials[k * grid + blk]
// for k < nv and of w . w in row nv (kUpdate only). A thread's row of the
// basis is loaded once, all loads in flight, and stays in registers; its nv
// sums run over all of its rows, so a work-group reduces each once.
template <int kGroups, bool kUpdate, bool kNt>
__global__ __launch_bounds__(kGmThreads, gm_resident(kGroups, kUpdate)) void gm_pass_kernel(
    int64_t n, const X *__restrict__ V, X *__restrict__ w, int nv, X *__restrict__ partials, const KState *st,
    GmState gs)
{
    if (st->flag != kRunning) return;
    constexpr int kMax = kGroups * kGmGroup;
    __shared__ double s_h[kMax];
    __shared__ X s_red[kGmThreads / kWave][kMax + 1];
    const X scale = kUpdate ? gs.s[nv - 1] : X(1);
    if (kUpdate) {
        if (threadIdx.x < kMax) s_h[threadIdx.x] = (int)threadIdx.x < nv ? st->dots[threadIdx.x] : 0.0;
        __syncthreads();
    }
    X acc[kMax], ww = X(0);
#pragma unroll
    for (int k = 0; k < kMax; ++k) acc[k] = X(0);
    const int64_t panels = (n + kGmThreads - 1) / kGmThreads;
    for (int64_t pb = blockIdx.x; pb < panels; pb += gridDim.x) {
        const X *__restrict__ P = V + pb * (gs.m + 1) * kGmThreads;  // uniform: one 32-bit lane offset
        const int64_t i = pb * kGmThreads + threadIdx.x;
        const bool in = i < n;
        const unsigned o = in ? threadIdx.x : 0u;
        X v[kMax];
        // a group's vectors past the last repeat it (their sums are not used)
#pragma unroll
        for (int k = 0; k < kMax; ++k) {
            const X *q = P + (k < nv ? k : nv - 1) * kGmThreads + o;
            v[k] = kNt ? ld_stream(q) : *q;
        }
        X wi = in ? w[i] : X(0);
        __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first use
        if (kUpdate) {
            wi *= scale;
#pragma unroll
            for (int k = 0; k < kMax; ++k) wi -= s_h[k] * v[k];
            if (in) w[i] = wi;
            else wi = X(0);
            ww += wi * wi;
        }
#pragma unroll
        for (int k = 0; k < kMax; ++k) acc[k] += v[k] * wi;
    }
    const int wid = threadIdx.x / kWave;
    int own = 0;
    const X sum = wave_sum_many<kMax>(acc, &own);
    if (own < kMax) s_red[wid][own] = sum;
    if (kUpdate) {
        const X t = wave_sum(ww);
        if (lane_id() == 0) s_red[wid][kMax] = t;
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < nv || (kUpdate && k == kMax)) {
        X t = X(0);
        for (int q = 0; q < kGmThreads / kWave; ++q) t += s_red[q][k];
        partials[(int64_t)(k < nv ? k : nv) * gridDim.x + blockIdx.x] = t;
    }
}

// Row k of the partials summed by work-group k. First pass: h_k = s_k s_{nv-1}
// (u_k . w). Second: h2_k = s_k (u_k . w') and, in row nv, ||w'|| (st->tmp[2]).
// st->dots[pass * kMaxDots + k] = h s_k, the coefficient of u_k.
__global__ __launch_bounds__(kGmThreads) void gm_dots_finish(const X *__restrict__ partials, int nb, int nv, int pass,
                                                            KState *st, GmState gs)
{
    if (st->flag != kRunning) return;
    __shared__ double s_sum[kGmThreads / kWave];
    const int k = blockIdx.x;
    const double t = block_sum_partials<X, kGmThreads>(partials + (int64_t)k * nb, nb, s_sum);
    if (threadIdx.x != 0) return;
    if (k == nv) {
        st->tmp[2] = sqrt(t);
        return;
    }
    const double h = pass == 0 ? gs.s[k] * (gs.s[nv - 1] * t) : gs.s[k] * t;
    (pass == 0 ? gs.h1 : gs.h2)[k] = h;
    st->dots[pass * kMaxDots + k] = h * gs.s[k];
}

// Third pass: u = (w' - sum_k dots[kMaxDots + k] u_k) / ||w'|| into column nv,
// z = M^{-1} u, partials of u . u. (A zero or non-finite ||w'|| leaves the
// scale out.)
__global__ __launch_bounds__(kGmThreads) void gm_last_pass_kernel(int64_t n, X *V, const X *__restrict__ w, int nv, int nt,
                                                                 const X *__restrict__ dinv, X *__restrict__ z,
                                                                 X *__restrict__ partials, const KState *st,
                                                                 GmState gs)
{
    if (st->flag != kRunning) return;
    __shared__ X s_red[kGmThreads / kWave];
    __shared__ double s_h[kMaxDots];
    if ((int)threadIdx.x < nv) s_h[threadIdx.x] = st->dots[kMaxDots + threadIdx.x];
    __syncthreads();
    const double wn = st->tmp[2];
    const X inv = wn > 0.0 && finite(1.0 / wn) ? 1.0 / wn : 1.0;
    X uu = X(0);
    const int64_t panels = (n + kGmThreads - 1) / kGmThreads;
    for (int64_t pb = blockIdx.x; pb < panels; pb += gridDim.x) {
        X *P = V + pb * (gs.m + 1) * kGmThreads;
        const int64_t i = pb * kGmThreads + threadIdx.x;
        if (i >= n) break;
        X wi = w[i];
        const X di = dinv ? dinv[i] : X(1);
        if (nt) {
#pragma unroll 8
            for (int k = 0; k < nv; ++k) wi -= s_h[k] * ld_stream(P + k * kGmThreads + threadIdx.x);
        } else {
#pragma unroll 8
            for (int k = 0; k < nv; ++k) wi -= s_h[k] * P[k * kGmThreads + threadIdx.x];
        }
        wi *= inv;
        P[nv * kGmThreads + threadIdx.x] = wi;
        z[i] = dinv ? wi * di : wi;
        uu += wi * wi;
    }
    X t[1] = {block_sum<X, kGmThreads>(uu, s_red)};
    write_partials<X, 1>(t, partials, gridDim.x, blockIdx.x);
}

// Arnoldi step finish: ||u||, Hessenberg column j, Givens rotations (staged
// in LDS, applied by one lane), the residual estimate and the cycle-end test
// (one work-group, fixed order).
__global__ __launch_bounds__(kGmThreads) void gm_step_finish(const X *__restrict__ partials, int nb, int j, KState *st,
                                                            GmState gs)
{
    if (st->flag != kRunning) return;
    __shared__ double s_sum[kGmThreads / kWave];
    __shared__ double s_h[kMaxDots], s_cs[kMaxDots], s_sn[kMaxDots];
    const int t = threadIdx.x;
    if (t <= j) s_h[t] = gs.h1[t] + gs.h2[t];
    if (t < j) {
        s_cs[t] = gs.cs[t];
        s_sn[t] = gs.sn[t];
    }
    const double un = sqrt(block_sum_partials<X, kGmThreads>(partials, nb, s_sum));
    const int m = gs.m;
    double *hj = gs.H + (int64_t)j * (m + 1);
    if (t == 0) {
        const double wn = st->tmp[2];
        const double hn = wn > 0.0 && finite(1.0 / wn) ? un * wn : un;
        double a = s_h[0];
        for (int i = 0; i < j; ++i) {  // previous rotations
            const double c = s_h[i + 1];
            s_h[i] = s_cs[i] * a + s_sn[i] * c;
            a = -s_sn[i] * a + s_cs[i] * c;
        }
        const double rho = hypot(a, hn);
        const double cs = a / rho, sn = hn / rho;
        gs.cs[j] = cs;
        gs.sn[j] = sn;
        s_h[j] = rho;
        hj[j + 1] = 0.0;
        const double gj = gs.g[j], gn = -sn * gj;
        gs.g[j + 1] = gn;
        gs.g[j] = cs * gj;
        gs.s[j + 1] = 1.0 / un;
        st->iters += 1;
        st->spmv_count += 1;
        st->jend = j + 1;
        st->rr = gn * gn;
        if (!finite(gn) || !finite(hn)) st->flag = kNonfinite;
        else if (gn * gn <= st->tol2 * st->bb || hn == 0.0 || st->iters >= st->maxit || j + 1 == m)
            st->flag = kCycleEnd;
    }
    __syncthreads();
    if (t <= j) hj[t] = s_h[t];
}

// y = H(0:jend,0:jend)^{-1} g (back substitution)
__global__ __launch_bounds__(kWave) void gm_solve_kernel(KState *st, GmState gs)
{
    // the wavefront stages the triangle and g in LDS, then one lane runs
    // the substitution (in the same order) on LDS instead of on dependent
    // global loads
    __shared__ double s_h[(kMaxDots - 1) * kMaxDots];
    __shared__ double s_y[kMaxDots];
    const int jend = st->jend, m = gs.m;
    for (int t = threadIdx.x; t < jend * jend; t += kWave) {
        const int k = t / jend, i = t % jend;
        if (i <= k) s_h[k * kMaxDots + i] = gs.H[(int64_t)k * (m + 1) + i];
    }
    for (int t = threadIdx.x; t < jend; t += kWave) s_y[t] = gs.g[t];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = jend - 1; i >= 0; --i) {
            double s = s_y[i];
            for (int k = i + 1; k < jend; ++k) s -= s_h[k * kMaxDots + i] * s_y[k];
            s_y[i] = s / s_h[i * kMaxDots + i];
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < jend; t += kWave) gs.y[t] = s_y[t];
}

// x += M^{-1} V y, V's columns being s_k u_k
__global__ __launch_bounds__(kGmThreads) void gm_xupdate_kernel(int64_t n, const X *__restrict__ V,
                                                               const X *__restrict__ dinv, X *__restrict__ x,
                                                               const KState *st, GmState gs)
{
    __shared__ double s_y[kMaxDots];
    const int jend = st->jend;
    if ((int)threadIdx.x < jend) s_y[threadIdx.x] = gs.y[threadIdx.x] * gs.s[threadIdx.x];
    __syncthreads();
    const X *__restrict__ P = V + (int64_t)blockIdx.x * (gs.m + 1) * kGmThreads;
    const int64_t i = (int64_t)blockIdx.x * kGmThreads + threadIdx.x;
    if (i >= n) return;
    X ul = X(0);
#pragma unroll 8
    for (int k = 0; k < jend; ++k) ul += s_y[k] * ld_stream(P + k * kGmThreads + threadIdx.x);
    x[i] += dinv ? ul * dinv[i] : ul;
}

__global__ void gm_zero_vec(int64_t n, X *__restrict__ x)
{
    const int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x;
    if (i < n) x[i] = X(0);
}

// ||b||^2 -> st->bb (zero rhs flagged)
__global__ __launch_bounds__(kVecThreads) void gm_bnorm_kernel(int64_t n, const X *__restrict__ b,
                                                              X *__restrict__ partials, KState *st)
{
    __shared__ X s_red[kVecThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kVecChunk;
    X acc = X(0);
#pragma unroll
    for (int u = 0; u < kVecItems; ++u) {
        const int64_t i = base + threadIdx.x + u * kVecThreads;
        if (i < n) acc += b[i] * b[i];
    }
    X v[1] = {block_sum<X, kVecThreads>(acc, s_red)};
    write_partials<X, 1>(v, partials, gridDim.x, blockIdx.x);
}

__global__ void gm_set_bb_kernel(KState *st)
{
    if (threadIdx.x == 0) {
        st->bb = st->tmp[0];
        if (!finite(st->bb)) st->flag = kNonfinite;
        else if (st->bb == 0.0) st->flag = kZeroRhs;
    }
}

struct GmBufs {
    X *V, *z, *q, *d, *dinv, *partials, *gmem;
    KState *st;
    int32_t *part;
};

// The pass kernel that holds nv vectors.
template <bool kUpdate, bool kNt>
static void gm_pass(int64_t n, const X *V, X *w, int nv, X *partials, const KState *st, const GmState &gs,
                    hipStream_t s)
{
    const unsigned gb = (unsigned)gm_blocks(n, nv, kUpdate);
#define SPX_GM_PASS(G)                                                                                      \
    case G: gm_pass_kernel<G, kUpdate, kNt><<<gb, kGmThreads, 0, s>>>(n, V, w, nv, partials, st, gs); break
    switch ((nv + kGmGroup - 1) / kGmGroup) {
        SPX_GM_PASS(1);
        SPX_GM_PASS(2);
        SPX_GM_PASS(3);
        SPX_GM_PASS(4);
        SPX_GM_PASS(5);
        SPX_GM_PASS(6);
        SPX_GM_PASS(7);
        SPX_GM_PASS(8);
        SPX_GM_PASS(9);
        SPX_GM_PASS(10);
        SPX_GM_PASS(11);
        SPX_GM_PASS(12);
        SPX_GM_PASS(13);
        SPX_GM_PASS(14);
        SPX_GM_PASS(15);
    default: gm_pass_kernel<16, kUpdate, kNt><<<gb, kGmThreads, 0, s>>>(n, V, w, nv, partials, st, gs); break;
    }
#undef SPX_GM_PASS
}

template <bool kUpdate>
static void gm_pass(int64_t n, const X *V, X *w, int nv, X *partials, const KState *st, const GmState &gs,
                    hipStream_t s)
{
    if (gm_streams(n, nv)) gm_pass<kUpdate, true>(n, V, w, nv, partials, st, gs, s);
    else gm_pass<kUpdate, false>(n, V, w, nv, partials, st, gs, s);
}

static GmBufs gm_carve(Carve &c, const spx_matrix &A, int precond, int m)
{
    const int64_t n = A.nrows;
    GmBufs w{};
    w.st = c.take<KState>(1);
    w.V = c.take<X>((int64_t)(m + 1) * gm_panels(n) * kGmThreads);
    w.q = c.take<X>(n);
    w.z = c.take<X>(n);
    w.d = precond ? c.take<X>(n) : nullptr;
    w.dinv = precond ? c.take<X>(n) : nullptr;
    const int64_t gb = gm_panels(n) < kGmBlocks ? gm_panels(n) : kGmBlocks;
    const int64_t slots = partial_slots(A) > (m + 2) * gb ? partial_slots(A) : (m + 2) * gb;
    w.partials = c.take<X>(slots);
    w.gmem = c.take<X>((int64_t)(m + 1) * m + 2 * (m + 1) + 5 * m);
    w.part = (A.fmt == SPX_CSR && A.csr_part == nullptr) ? c.take<int32_t>(csr_partition_bytes(A.nnz) / 4) : nullptr;
    return w;
}

size_t gmres_workspace(const spx_matrix &A, int precond, int restart)
{
    Carve c(nullptr, 0);
    (void)gm_carve(c, A, precond, restart);
    return c.off + 256;
}

spx_status gmres_run(const spx_matrix &A_in, const double *b, double *x, const SolveSpec &sp, void *ws,
                     size_t ws_bytes, spx_solve_info *info, hipStream_t user_stream)
{
    const int m = sp.restart;
    SPX_REQUIRE(m >= 1 && m <= kMaxDots - 2, SPX_ERR_ARG, "gmres: restart must be in [1, %d]", kMaxDots - 2);
    SolveEnv *env = nullptr;
    SPX_CHECK(solve_env(&env));
    hipStream_t s = env->stream;
    const int64_t n = A_in.nrows;
    Carve c(ws, ws_bytes);
    GmBufs w = gm_carve(c, A_in, sp.precond, m);
    SPX_REQUIRE(c.fits(), SPX_ERR_ARG, "gmres: workspace of %zu bytes is too small (need %zu)", ws_bytes,
                gmres_workspace(A_in, sp.precond, m));
    spx_matrix A = A_in;
    *info = spx_solve_info{};
    X *gv0 = w.gmem + (m + 1) * m;  // behind H: g, s, then cs, sn, y, h1, h2
    X *gm0 = gv0 + 2 * (m + 1);
    GmState gs{m, w.gmem, gv0, gm0, gm0 + m, gm0 + 2 * m, gv0 + (m + 1), gm0 + 3 * m, gm0 + 4 * m};

    SPX_HIP(hipEventRecord(env->join, user_stream));
    SPX_HIP(hipStreamWaitEvent(s, env->join, 0));
    SPX_HIP(hipEventRecord(env->ev0, s));
    if (w.part) {
        SPX_CHECK(csr_partition_launch(A, w.part, s));
        A.csr_part = w.part;
    }
    SPX_CHECK(state_init(w.st, sp.tol, sp.maxit, s));
    KState hs;
    if (sp.precond) {
        SPX_CHECK((jacobi_setup<double, double>(A, w.d, w.dinv, w.st, s)));
        SPX_CHECK(read_state(env, w.st, &hs));
        if (hs.flag != kRunning) {
            set_error("gmres: zero, missing or non-finite diagonal entry");
            return SPX_ERR_ZERO_DIAG;
        }
    }
    const unsigned gv = (unsigned)vec_blocks(n);
    const unsigned ge = (unsigned)ceil_div(n, kVecThreads);
    if (sp.x0_zero) gm_zero_vec<<<ge, kVecThreads, 0, s>>>(n, x);
    gm_bnorm_kernel<<<gv, kVecThreads, 0, s>>>(n, b, w.partials, w.st);
    SPX_LAUNCHED();
    SPX_CHECK(launch_finish<X>(w.partials, gv, 1, w.st, kOpNorm2, s));
    gm_set_bb_kernel<<<1, 64, 0, s>>>(w.st);
    SPX_LAUNCHED();

    GraphGuard graph;
    const unsigned gp = (unsigned)gm_panels(n), gl = gp < (unsigned)kGmBlocks ? gp : (unsigned)kGmBlocks;
    auto cycle = [&]() -> spx_status {
        for (int j = 0; j < m; ++j) {
            const int nv = j + 1;
            const int gd = (int)gm_blocks(n, nv, false), gu = (int)gm_blocks(n, nv, true);
            SPX_CHECK((spmv_st<double, double>(A, w.z, w.q, w.st, s)));
            gm_pass<false>(n, w.V, w.q, nv, w.partials, w.st, gs, s);
            gm_dots_finish<<<nv, kGmThreads, 0, s>>>(w.partials, gd, nv, 0, w.st, gs);
            gm_pass<true>(n, w.V, w.q, nv, w.partials, w.st, gs, s);
            gm_dots_finish<<<nv + 1, kGmThreads, 0, s>>>(w.partials, gu, nv, 1, w.st, gs);
            gm_last_pass_kernel<<<gl, kGmThreads, 0, s>>>(n, w.V, w.q, nv, gm_streams(n, nv), w.dinv, w.z,
                                                           w.partials, w.st, gs);
            gm_step_finish<<<1, kGmThreads, 0, s>>>(w.partials, (int)gl, j, w.st, gs);
            SPX_LAUNCHED();
        }
        return SPX_OK;
    };
    spx_status status = SPX_OK;
    double true2 = 0.0;
    while (true) {
        // true residual r = b - A x into z
        SPX_CHECK(spmv_dispatch(A, x, w.q, 1.0, 0.0, s));
        SPX_CHECK(residual_norm<double>(n, b, w.q, w.z, w.partials, w.st, s));
        SPX_CHECK(read_state(env, w.st, &hs));
        true2 = hs.tmp[0];
        if (hs.flag == kZeroRhs) {
            gm_zero_vec<<<ge, kVecThreads, 0, s>>>(n, x);
            SPX_LAUNCHED();
            true2 = 0.0;
            status = SPX_OK;
            break;
        }
        if (hs.flag == kNonfinite || !std::isfinite(true2)) {
            status = SPX_ERR_NONFINITE;
            set_error("gmres: non-finite residual");
            break;
        }
        if (true2 <= hs.tol2 * hs.bb) {
            status = SPX_OK;
            break;
        }
        if (hs.iters >= sp.maxit) {
            status = SPX_ERR_NOT_CONVERGED;
            set_error("gmres: no convergence in %d Arnoldi steps", sp.maxit);
            break;
        }
        gm_cycle_init_kernel<<<gp, kGmThreads, 0, s>>>(n, w.dinv, w.V, w.z, w.st, gs);
        SPX_LAUNCHED();
        if (graph.exec == nullptr) SPX_CHECK(capture_graph(s, &graph.exec, cycle));
        SPX_HIP(hipGraphLaunch(graph.exec, s));
        gm_solve_kernel<<<1, 64, 0, s>>>(w.st, gs);
        gm_xupdate_kernel<<<gp, kGmThreads, 0, s>>>(n, w.V, w.dinv, x, w.st, gs);
        SPX_LAUNCHED();
        SPX_CHECK(read_state(env, w.st, &hs));
        info->outer_iters += 1;
        if (hs.flag == kNonfinite) {
            status = SPX_ERR_NONFINITE;
            set_error("gmres: non-finite residual");
            break;
        }
    }
    SPX_HIP(hipEventRecord(env->ev1, s));
    SPX_HIP(hipEventSynchronize(env->ev1));
    float ms = 0.f;
    SPX_HIP(hipEventElapsedTime(&ms, env->ev0, env->ev1));
    info->status = status;
    info->iters = hs.iters;
    info->spmv_count = hs.spmv_count + info->outer_iters + 1;
    info->relres_recursive = hs.bb > 0 ? sqrt(hs.rr / hs.bb) : 0.0;
    info->relres_true = hs.bb > 0 ? sqrt(true2 / hs.bb) : 0.0;
    info->device_ms = ms;
    SPX_HIP(hipEventRecord(env->join, s));
    SPX_HIP(hipStreamWaitEvent(user_stream, env->join, 0));
    return status;
}

}  // namespace spx
