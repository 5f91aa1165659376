// Preconditioned conjugate gradients in float64 (the Krylov solver of the
// paper's symmetric positive definite experiments, Sections 9 and 10), for
// use with the symmetric GS2 (SGS2) preconditioner.  Textbook recurrences;
// the recurrence residual decides when to stop, the true residual is then
// checked and the iteration restarts from it if it has drifted.  Every
// scalar (alpha, beta, the stopping test) is formed on the device; the host
// enqueues iterations in chunks and synchronises once per chunk, kernels
// return at once after the stopping test has fired.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <new>

#include "gs2_internal.hpp"
#include "sella.hpp"

namespace gs2 {

constexpr int CT = 256;  // threads per workgroup
constexpr int CRB = 1024; // rows per workgroup of the vector kernels

struct CState {
    int it, done, maxit, status, flag; // flag: FILL_*
    double bnorm, rtol, rz, pq, rr, beta;
};

struct CgWork {
    int64_t n = 0;
    int nb = 0;
    void *mem = nullptr; // one allocation behind the device arrays
    double *r = nullptr, *z = nullptr, *p = nullptr, *q = nullptr, *part = nullptr, *part2 = nullptr;
    Product prod; // with a handle: the solver's copy of A
    CState *st = nullptr, *hst = nullptr;
};

void free_cg_work(CgWork *w)
{
    if (!w) return;
    sella_free(w->prod.A);
    if (w->mem) (void)hipFree(w->mem);
    if (w->hst) (void)hipHostFree(w->hst);
    delete w;
}

static int alloc_cg(CgWork **out, int64_t n)
{
    CgWork *w = new (std::nothrow) CgWork;
    if (!w) return GS2_ERR_NOMEM;
    w->n = n;
    w->nb = (int)std::max<int64_t>(1, (n + CRB - 1) / CRB);
    const size_t N = (size_t)std::max<int64_t>(n, 1), v = aligned(8 * N), np = aligned(8 * (N / CT + 2));
    int st = GS2_OK;
    if (hipMalloc(&w->mem, 4 * v + 2 * np + aligned(sizeof(CState)) + pattern_dev_bytes()) != hipSuccess) {
        st = GS2_ERR_NOMEM;
    } else {
        char *m = (char *)w->mem;
        w->r = (double *)m;
        w->z = (double *)(m + v);
        w->p = (double *)(m + 2 * v);
        w->q = (double *)(m + 3 * v);
        w->part = (double *)(m + 4 * v);
        w->part2 = (double *)(m + 4 * v + np);
        w->st = (CState *)(m + 4 * v + 2 * np);
        w->prod.pat = (PatternDev *)(m + 4 * v + 2 * np + aligned(sizeof(CState)));
        w->prod.in = w->z;
        w->prod.out = w->q;
        w->prod.part = w->part;
    }
    if (st == GS2_OK && hipHostMalloc((void **)&w->hst, sizeof(CState), hipHostMallocDefault) != hipSuccess)
        st = GS2_ERR_NOMEM;
    if (st != GS2_OK) {
        free_cg_work(w);
        return st;
    }
    *out = w;
    return GS2_OK;
}

__device__ __forceinline__ double cg_block_sum(double v, double *red)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) red[threadIdx.x / WAVE] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < CT / WAVE; ++i) s += red[i];
    return s;
}

// out = b - A x (when b != NULL) or out = A x, with partial sums of
// out.x2 (x2 = out when x2 == NULL).  K lanes per row.
template <int K>
__global__ __launch_bounds__(CT) void k_cg_spmv(int64_t n, const int32_t *__restrict__ rp,
                                                const int32_t *__restrict__ ci, const double *__restrict__ va,
                                                const double *__restrict__ x, const double *__restrict__ b,
                                                double *__restrict__ out, const double *__restrict__ x2,
                                                const int *__restrict__ stop, double *__restrict__ part)
{
    __shared__ double red[CT / WAVE];
    if (stop && *stop) return;
    const int64_t r0 = (int64_t)blockIdx.x * CRB;
    const int t = threadIdx.x, q = t & (K - 1);
    constexpr int RPP = CT / K;
    double s = 0.0;
    for (int pass = 0; pass < CRB / RPP; ++pass) {
        const int64_t row = r0 + pass * RPP + t / K;
        double acc = 0.0;
        if (row < n) {
            const int bb = rp[row], e = rp[row + 1];
            for (int p = bb + q; p < e; p += K) acc += va[p] * x[ci[p]];
        }
        acc = group_sum<K>(acc);
        if (q == 0 && row < n) {
            const double o = b ? b[row] - acc : acc;
            out[row] = o;
            s += o * (x2 ? x2[row] : o);
        }
    }
    s = cg_block_sum(s, red);
    if (t == 0) part[blockIdx.x] = s;
}

// sum of a thread's partials b = threadIdx.x, + CT, ..., eight loads in flight
__device__ __forceinline__ double cg_part_sum(const double *__restrict__ part, int nb)
{
    constexpr int U = 8;
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.0;
    for (int b0 = threadIdx.x; b0 < nb; b0 += CT * U)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + u * CT;
            acc[u] += b < nb ? part[b] : 0.0;
        }
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) s += acc[u];
    return s;
}

// sum of the partials into *dst
__global__ __launch_bounds__(CT) void k_cg_reduce(const double *__restrict__ part, int nb, const int *__restrict__ stop,
                                                  double *__restrict__ dst)
{
    __shared__ double red[CT / WAVE];
    if (stop && *stop) return;
    const double s = cg_block_sum(cg_part_sum(part, nb), red);
    if (threadIdx.x == 0) *dst = s;
}

// what closes an iteration, in one launch: ||r||^2 from the update's partials
// with the stopping test, and r.z from the dot's with beta
__global__ __launch_bounds__(CT) void k_cg_close(const double *__restrict__ rpart, int nr,
                                                 const double *__restrict__ zpart, int nz, CState *__restrict__ st)
{
    __shared__ double red[CT / WAVE];
    if (st->done) return;
    const double pr = cg_part_sum(rpart, nr), pz = cg_part_sum(zpart, nz);
    const double rr = cg_block_sum(pr, red);
    const double rz = cg_block_sum(pz, red);
    if (threadIdx.x != 0) return;
    st->rr = rr;
    st->it += 1;
    if (!isfinite(rr)) {
        st->status = GS2_ERR_NONFINITE;
        st->done = 1;
    } else if (sqrt(rr) <= st->rtol * st->bnorm || st->it >= st->maxit) {
        st->done = 1;
    }
    st->beta = rz / st->rz;
    st->rz = rz;
}

// x += alpha p, r -= alpha q (alpha = rz / pq), partial ||r||^2
__global__ __launch_bounds__(CT) void k_cg_update(int64_t n, const double *__restrict__ p,
                                                  const double *__restrict__ q, double *__restrict__ x,
                                                  double *__restrict__ r, const CState *__restrict__ st,
                                                  double *__restrict__ part)
{
    __shared__ double red[CT / WAVE];
    if (st->done) return;
    const double alpha = st->rz / st->pq;
    const int64_t r0 = (int64_t)blockIdx.x * CRB;
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < CRB / CT; ++u) {
        const int64_t i = r0 + threadIdx.x + u * CT;
        if (i < n) {
            x[i] += alpha * p[i];
            const double ri = r[i] - alpha * q[i];
            r[i] = ri;
            s += ri * ri;
        }
    }
    s = cg_block_sum(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// partial r.z
__global__ __launch_bounds__(CT) void k_cg_dot(int64_t n, const double *__restrict__ a, const double *__restrict__ b,
                                               const CState *__restrict__ st, double *__restrict__ part)
{
    __shared__ double red[CT / WAVE];
    if (st && st->done) return;
    const int64_t r0 = (int64_t)blockIdx.x * CRB;
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < CRB / CT; ++u) {
        const int64_t i = r0 + threadIdx.x + u * CT;
        if (i < n) s += a[i] * b[i];
    }
    s = cg_block_sum(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// p = z + beta p  (beta_mode 0: p = z)
__global__ void k_cg_p(int64_t n, const double *__restrict__ z, double *__restrict__ p,
                       const CState *__restrict__ st, int beta_mode)
{
    if (st->done) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    p[i] = beta_mode ? z[i] + st->beta * p[i] : z[i];
}

__global__ void k_cg_copy(int64_t n, const double *__restrict__ a, double *__restrict__ b, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = a[i];
}

__global__ void k_cg_start(CState *__restrict__ st, int maxit_total, double rtol)
{
    if (threadIdx.x) return;
    st->done = 0;
    st->maxit = maxit_total;
    st->rtol = rtol;
}

static int cg_lanes(const gs2_csr &A)
{
    const double avg = A.n ? (double)A.nnz / (double)A.n : 1.0;
    return avg <= 8.0 ? 4 : avg <= 16.0 ? 8 : avg <= 32.0 ? 16 : avg <= 64.0 ? 32 : 64;
}

#define GS2_CG_DISPATCH(K, kern, grid, ...)                                  \
    do {                                                                     \
        switch (K) {                                                         \
        case 4: kern<4><<<grid, CT, 0, s>>>(__VA_ARGS__); break;             \
        case 8: kern<8><<<grid, CT, 0, s>>>(__VA_ARGS__); break;             \
        case 16: kern<16><<<grid, CT, 0, s>>>(__VA_ARGS__); break;           \
        case 32: kern<32><<<grid, CT, 0, s>>>(__VA_ARGS__); break;           \
        default: kern<64><<<grid, CT, 0, s>>>(__VA_ARGS__); break;           \
        }                                                                    \
    } while (0)

static int cg_impl(const gs2_csr &A, const double *b, double *x, double rtol, int maxit, int kind, gs2_handle *P,
                   gs2_solve_info *info, hipStream_t s)
{
    const int64_t n = A.n;
    CgWork *own = nullptr, *W = nullptr;
    if (P) {
        if (!P->h.cw || P->h.cw->n != n) {
            if (P->h.cw) free_cg_work(P->h.cw);
            P->h.cw = nullptr;
            GS2_TRY(alloc_cg(&P->h.cw, n));
        }
        W = P->h.cw;
    } else {
        GS2_TRY(alloc_cg(&own, n));
        W = own;
    }
    struct Guard {
        CgWork *w;
        gs2_handle *P;
        ~Guard()
        {
            if (w) free_cg_work(w);
            if (P) P->h.stop = nullptr;
        }
    } guard{own, P};
    CState *st = W->st;
    if (P) P->h.stop = &st->done;
    const int nb = W->nb, K = cg_lanes(A);
    const unsigned gN = (unsigned)nb, gE = (unsigned)((n + 255) / 256);
    auto prec = [&](const double *v, double *z) -> int {
        switch (kind) {
        case GS2_PREC_GS2: return apply_gs2(P->h, v, z, s);
        case GS2_PREC_JR: return apply_jr(P->h, P->h.sweeps, P->h.omega, v, z, s);
        case GS2_PREC_GS_TRISOLVE: return apply_trisolve(P->h, P->h.variant, P->h.omega, v, z, s);
        case GS2_PREC_MTGS: return apply_mtgs(P->h, P->h.variant, P->h.omega, v, z, s);
        default: k_cg_copy<<<gE, 256, 0, s>>>(n, v, z, &st->done); return GS2_OK;
        }
    };
    auto read_state = [&]() -> int {
        GS2_TRY_HIP(hipMemcpyAsync(W->hst, st, sizeof(CState), hipMemcpyDeviceToHost, s));
        GS2_TRY_HIP(hipStreamSynchronize(s));
        return GS2_OK;
    };
    // ||b||, initial state
    {
        // staged in the pinned mirror (no copy from it is in flight here)
        CState init{};
        init.rtol = rtol;
        init.maxit = maxit;
        *W->hst = init;
        GS2_TRY_HIP(hipMemcpyAsync(st, W->hst, sizeof(CState), hipMemcpyHostToDevice, s));
    }
    // With a handle, which lives on, the products run on a copy of A in the
    // layout that suits it (as gmres_solve's): 20 against 46 us per
    // product on a 120^3 7-point matrix, 77 against 89 us per iteration on 300,000
    // rows of 15 random entries.  On the CSR arrays where there is no
    // handle, no memory for a copy, rows that are no longer strictly sorted, or a
    // few rows much longer than the others (prepare_product).
    bool copied = P != nullptr;
    auto copy = [&]() -> int {
        const int e = prepare_product(W->prod, A, P->h.spmv_fmt, s, &st->flag, false);
        if (e == GS2_OK) copied = W->prod.built();
        if (e != GS2_ERR_NOMEM) return e;
        (void)hipGetLastError();
        copied = false;
        return GS2_OK;
    };
    if (copied) GS2_TRY(copy());
    k_cg_dot<<<gN, CT, 0, s>>>(n, b, b, nullptr, W->part);
    k_cg_reduce<<<1, CT, 0, s>>>(W->part, nb, nullptr, &st->bnorm);
    GS2_TRY_HIP(hipGetLastError());
    GS2_TRY(read_state());
    if (copied && W->hst->flag == FILL_CHANGED) {
        W->prod.fmt_req = -1;
        W->hst->flag = 0;
        GS2_TRY_HIP(hipMemcpyAsync(&st->flag, &W->hst->flag, sizeof(int), hipMemcpyHostToDevice, s));
        GS2_TRY(copy());
        GS2_TRY(read_state());
    }
    if (W->hst->flag) copied = false;
    // what an iteration reads beside the copy: six vectors and the triangles
    double beside = 48.0 * n;
    if (P && kind != GS2_PREC_NONE)
        beside += P->h.fmt == FMT_DIA ? P->h.DL.stored_bytes() + P->h.DU.stored_bytes()
                                      : P->h.L.stored_bytes() + P->h.U.stored_bytes();
    const double spmv_b = copied ? sella_bytes(W->prod.A) : 12.0 * (double)A.nnz + 4.0 * (n + 1) + 16.0 * n;
    const double bn2 = W->hst->bnorm;
    if (!std::isfinite(bn2)) return GS2_ERR_NONFINITE;
    if (bn2 == 0.0) {
        GS2_TRY_HIP(hipMemsetAsync(x, 0, sizeof(double) * n, s));
        GS2_TRY_HIP(hipStreamSynchronize(s));
        info->converged = 1;
        return GS2_OK;
    }
    const double bnorm = std::sqrt(bn2);
    {
        CState init{}; // the mirror was last filled by read_state, which synchronised
        init.bnorm = bnorm;
        init.rtol = rtol;
        init.maxit = maxit;
        *W->hst = init;
        GS2_TRY_HIP(hipMemcpyAsync(st, W->hst, sizeof(CState), hipMemcpyHostToDevice, s));
    }
    int status = GS2_OK, runs = 0;
    for (;;) {
        // true residual r = b - A x
        int np = nb;
        {
            Prof pr(s, PK_TRUE_RESID, spmv_b + 8.0 * n);
            if (copied) np = product_resid(W->prod, x, b, W->r, W->part, s);
            else
                GS2_CG_DISPATCH(K, k_cg_spmv, gN, n, A.rowptr, A.colind, A.val, x, b, W->r, nullptr, nullptr, W->part);
        }
        k_cg_reduce<<<1, CT, 0, s>>>(W->part, np, nullptr, &st->rr);
        GS2_TRY_HIP(hipGetLastError());
        GS2_TRY(read_state());
        const CState hs = *W->hst;
        if (hs.status != GS2_OK) { status = hs.status; break; }
        const double rel = std::sqrt(hs.rr) / bnorm;
        info->relres = rel;
        info->iterations = hs.it;
        if (!std::isfinite(rel)) { status = GS2_ERR_NONFINITE; break; }
        if (rel <= rtol) { info->converged = 1; break; }
        if (hs.it >= maxit) { status = GS2_NOT_CONVERGED; break; }
        if (runs++ > 0) info->restarts++;
        k_cg_start<<<1, 64, 0, s>>>(st, maxit, rtol);
        // z = M^-1 r, p = z, rz = r.z
        GS2_TRY(prec(W->r, W->z));
        k_cg_dot<<<gN, CT, 0, s>>>(n, W->r, W->z, st, W->part);
        k_cg_reduce<<<1, CT, 0, s>>>(W->part, nb, nullptr, &st->rz);
        k_cg_p<<<gE, 256, 0, s>>>(n, W->z, W->p, st, 0);
        int chunk = 8;
        for (;;) {
            for (int c = 0; c < chunk; ++c) {
                int np = nb;
                {   // q = A p, p.q
                    Prof pr(s, PK_SPMV_DOT, spmv_b);
                    if (copied) np = product_dot(W->prod, W->p, W->q, &st->done, W->part, beside, s);
                    else
                        GS2_CG_DISPATCH(K, k_cg_spmv, gN, n, A.rowptr, A.colind, A.val, W->p, nullptr, W->q, W->p,
                                        &st->done, W->part);
                }
                k_cg_reduce<<<1, CT, 0, s>>>(W->part, np, &st->done, &st->pq);
                {
                    Prof pr(s, PK_CGS, 48.0 * n);
                    k_cg_update<<<gN, CT, 0, s>>>(n, W->p, W->q, x, W->r, st, W->part2);
                }
                GS2_TRY(prec(W->r, W->z));
                k_cg_dot<<<gN, CT, 0, s>>>(n, W->r, W->z, st, W->part);
                k_cg_close<<<1, CT, 0, s>>>(W->part2, nb, W->part, nb, st);
                {
                    Prof pr(s, PK_SCALE, 24.0 * n);
                    k_cg_p<<<gE, 256, 0, s>>>(n, W->z, W->p, st, 1);
                }
            }
            GS2_TRY_HIP(hipGetLastError());
            GS2_TRY(read_state());
            if (W->hst->done) break;
            chunk = std::min(chunk * 2, 64);
        }
    }
    return status;
}

} // namespace gs2

using namespace gs2;

extern "C" int cg_solve(const gs2_csr *A, const double *b, double *x, double rtol, int maxit, int prec_kind,
                        gs2_handle *prec, gs2_solve_info *info, void *stream)
{
    gs2_solve_info local;
    gs2_solve_info *inf = info ? info : &local;
    std::memset(inf, 0, sizeof(*inf));
    const auto t0 = std::chrono::steady_clock::now();
    int st;
    if (!A || A->n <= 0 || A->n >= (int64_t(1) << 31) - 1 || !A->rowptr || !A->colind || !A->val || !b || !x ||
        !(rtol >= 0.0) || maxit < 0 || prec_kind < GS2_PREC_NONE || prec_kind > GS2_PREC_MTGS ||
        (prec_kind != GS2_PREC_NONE && !prec) || (prec && prec->h.n != A->n)) {
        st = GS2_ERR_ARG;
    } else if ((prec_kind == GS2_PREC_GS_TRISOLVE && prec->h.nlev_l == 0) ||
               (prec_kind == GS2_PREC_MTGS && prec->h.ncolors == 0)) {
        st = GS2_ERR_NO_LEVELS;
    } else {
        try {
            st = cg_impl(*A, b, x, rtol, maxit, prec_kind, prec, inf, (hipStream_t)stream);
        } catch (const std::bad_alloc &) {
            st = GS2_ERR_NOMEM;
        } catch (...) {
            st = GS2_ERR_HIP;
        }
    }
    inf->status = st;
    inf->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return st;
}
