// The device-side state of a GMRES restart cycle and the serial work that
// closes an Arnoldi step of the delayed reorthogonalisation.  Shared by the
// Krylov kernels and by the first preconditioner pass of the next step,
// which runs that work in one extra workgroup (k_inner, k_first_jr).
#pragma once

#include <cstddef>

#include "gs2_internal.hpp"

namespace gs2 {

constexpr int MAXM = 128; // longest restart supported
constexpr int KT = 256;   // threads per workgroup of the Krylov kernels

struct GState {
    int j, done, kk, status;
    int maxsteps, pad0, pad1, pad2;
    double bnorm, beta, rtol, inv;
    double hA[MAXM + 2], hB[MAXM + 2], nrm[2];
    double g[MAXM + 2], cs[MAXM], sn[MAXM], y[MAXM];
    // delayed CGS2: scalars of the current step and the tentative column
    double bb, dd, wn2, nu, inv_alpha, e;
    double ht[MAXM + 2];
    // scale of the stored preconditioned vector of each step: step j works on
    // the unnormalised tentative vector, z_j = zs[j] * (stored Z column j)
    double zs[MAXM + 2];
    // last, so that everything before it can be staged in LDS (8.5 KB)
    double H[(MAXM + 1) * MAXM]; // H[k * MAXM + col], upper triangle R after rotations
};
constexpr int GSTATE_SMALL_WORDS = (int)(offsetof(GState, H) / 8);
static_assert(offsetof(GState, H) % 8 == 0, "the staged part of the state is whole 8-byte words");

// Sum of p[b] over this thread's b = threadIdx.x, + KT, ... < cnt.  Eight
// loads are in flight at once (a plain strided loop waits for each load
// before the next: one memory latency per partial); the eight running sums
// are added in a fixed order.
__device__ __forceinline__ double strided_sum(const double *__restrict__ p, int cnt)
{
    constexpr int U = 8;
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.0;
    for (int b0 = threadIdx.x; b0 < cnt; b0 += KT * U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + u * KT;
            acc[u] += b < cnt ? p[b] : 0.0;
        }
    }
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) s += acc[u];
    return s;
}

// Sum of one value per thread over the workgroup (KT threads); result valid
// in thread 0.  Starts and ends with a barrier.
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    const int wv = threadIdx.x / WAVE;
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) red[wv] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < KT / WAVE; ++i) s += red[i];
    return s;
}

// Orders a wavefront's LDS accesses before and after (its lanes run in step).
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// (one lane) Apply rotations 0..jc-1 to col (jc+1 entries used).  The entry
// carried from one rotation to the next stays in a register, so the chain
// is two multiply-adds per rotation; a block's loads are issued before its
// first rotation.  The fused operations are written out here and below, so
// that every kernel these are part of rounds alike.
__device__ __forceinline__ void apply_rotations(const double *cs, const double *sn, double *col, int jc)
{
    constexpr int U = 4;
    double carry = col[0];
    for (int k0 = 0; k0 < jc; k0 += U) {
        double c[U], s[U], x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int k = k0 + q < jc ? k0 + q : jc - 1;
            c[q] = cs[k];
            s[q] = sn[k];
            x[q] = col[k + 1];
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (k0 + q < jc) {
                col[k0 + q] = fma(c[q], carry, s[q] * x[q]);
                carry = fma(-s[q], carry, c[q] * x[q]);
            }
    }
    col[jc] = carry;
}

// (one wavefront) Apply the committed rotations 0..jc-1 of the state ls (in
// LDS) to col (jc+2 entries), form rotation jc, store column jc of R into H
// (row stride ldh) and advance the residual recurrence g.  col is complete
// on entry (wave_fence).
__device__ inline bool commit_column(GState *ls, double *__restrict__ H, int ldh, double *col, int jc)
{
    const int ln = threadIdx.x & (WAVE - 1);
    if (ln == 0) apply_rotations(ls->cs, ls->sn, col, jc);
    wave_fence();
    const double rho = hypot(col[jc], col[jc + 1]);
    if (!isfinite(rho)) {
        if (ln == 0) ls->status = GS2_ERR_NONFINITE;
        return false;
    }
    if (rho == 0.0) {
        if (ln == 0) ls->status = GS2_BREAKDOWN_EXACT;
        return false;
    }
    const double c = col[jc] / rho, sn = col[jc + 1] / rho;
    for (int k = ln; k < jc; k += WAVE) H[k * ldh + jc] = col[k];
    if (ln == 0) {
        H[jc * ldh + jc] = rho;
        ls->cs[jc] = c;
        ls->sn[jc] = sn;
        const double gj = ls->g[jc];
        ls->g[jc + 1] = -sn * gj;
        ls->g[jc] = c * gj;
    }
    wave_fence();
    return true;
}

// Reorthogonalisation scalars of u from the reduced sums of pass 1:
// alpha^2 = u.u - |a|^2 and e = (u.w - a.c)/alpha (alpha = 1, e = u.w at
// j = 0).  as/cs_ hold a and c in LDS; the sums run in one wavefront in a
// fixed order, so every workgroup that calls this gets the same bits.
// Returns false when u has fallen into span(Q) (or alpha^2 is not finite).
__device__ inline bool reorth_scalars(const GState *st, int j, const double *as, const double *cs_, double *sc,
                               double *alpha, double *e, double *a2)
{
    const int t = threadIdx.x, ln = t & (WAVE - 1);
    if (t < WAVE) {
        double aa = 0.0, ac = 0.0;
        for (int k = ln; k < j; k += WAVE) {
            aa = fma(as[k], as[k], aa);
            ac = fma(as[k], cs_[k], ac);
        }
        aa = wave_sum(aa);
        ac = wave_sum(ac);
        if (ln == 0) {
            sc[0] = aa;
            sc[1] = ac;
        }
    }
    __syncthreads();
    *a2 = st->bb - sc[0];
    const bool ok = j == 0 || (isfinite(*a2) && *a2 > 0.0);
    *alpha = j == 0 ? 1.0 : sqrt(*a2);
    *e = j == 0 ? st->dd : (st->dd - sc[1]) / *alpha;
    return ok;
}

// (one wavefront) The step's serial work on the state ls (in LDS): correct
// and commit column j-1 ([ht + nu a; nu alpha]) now that u's
// reorthogonalisation is known, store the new tentative column [c, e], take
// ||w'||^2 = tot, form the tentative rotation of column j and the residual
// estimate, and either stop the cycle or advance j (the next tentative vector
// keeps its scale 1/||w'|| in zs[j+1]).  When u fell into span(Q) (!ok) the
// cycle ends on the tentative column j-1.  Only the two chains of rotations
// run in one lane; with all of it there, the work took 5 us at 30 columns.
__device__ inline void dcgs_finish_wave(GState *ls, double *__restrict__ H, int ldh, double *col, bool ok,
                                        double alpha, double e, double a2, double tot)
{
    const int ln = threadIdx.x & (WAVE - 1);
    const bool one = ln == 0;
    const int j = ls->j;
    const double nu_prev = ls->nu;
    if (!ok) {
        int kk = j - 1;
        if (!isfinite(a2)) {
            if (one) ls->status = GS2_ERR_NONFINITE;
        } else {
            for (int k = ln; k < j; k += WAVE) col[k] = ls->ht[k];
            if (one) col[j] = nu_prev;
            wave_fence();
            if (commit_column(ls, H, ldh, col, j - 1)) kk = j;
        }
        if (one) {
            ls->kk = kk;
            ls->done = 1;
        }
        return;
    }
    if (j > 0) {
        for (int k = ln; k < j; k += WAVE) col[k] = fma(nu_prev, ls->hA[k], ls->ht[k]);
        if (one) col[j] = nu_prev * alpha;
        wave_fence();
        if (!commit_column(ls, H, ldh, col, j - 1)) {
            if (one) {
                ls->kk = j - 1;
                ls->done = 1;
            }
            return;
        }
    }
    // tentative column j: [c, e; ||w'||]
    const double nu = sqrt(tot);
    for (int k = ln; k < j; k += WAVE) {
        const double c = ls->hB[k];
        ls->ht[k] = c;
        col[k] = c;
    }
    if (one) {
        ls->inv_alpha = 1.0 / alpha;
        ls->e = e;
        ls->ht[j] = e;
        ls->nu = nu;
        col[j] = e;
        col[j + 1] = nu;
    }
    wave_fence();
    if (one) apply_rotations(ls->cs, ls->sn, col, j);
    wave_fence();
    const double rho = hypot(col[j], col[j + 1]);
    if (!isfinite(rho) || !isfinite(nu)) {
        if (one) {
            ls->status = GS2_ERR_NONFINITE;
            ls->done = 1;
            ls->kk = j;
        }
        return;
    }
    const double est = rho > 0.0 ? fabs(col[j + 1] / rho * ls->g[j]) : 0.0;
    const bool breakdown = nu <= 1e-14 * sqrt(ls->wn2);
    if (est <= ls->rtol * ls->bnorm || breakdown || j + 1 >= ls->maxsteps) {
        wave_fence();
        for (int k = ln; k < j; k += WAVE) col[k] = ls->ht[k];
        if (one) {
            col[j] = e;
            col[j + 1] = nu;
        }
        wave_fence();
        const bool good = commit_column(ls, H, ldh, col, j);
        if (one) {
            ls->kk = good ? j + 1 : j;
            ls->done = 1;
        }
    } else if (one) {
        ls->kk = j + 1;
        ls->inv = 1.0 / nu;
        ls->zs[j + 1] = 1.0 / nu;
        ls->j = j + 1;
    }
}

// The step's serial work (one workgroup, KT threads).  It is latency-bound:
// the whole workgroup stages the state (all but H) in LDS together with the
// partial sums, so one round trip to memory precedes the serial work of one
// wavefront, and writes it back.
__device__ __forceinline__ void dcgs_finish_block(const double *__restrict__ part, int nb, GState *__restrict__ st)
{
    __shared__ unsigned long long sw[GSTATE_SMALL_WORDS];
    __shared__ double col[MAXM + 2], red[KT / WAVE], sc[2];
    GState *ls = reinterpret_cast<GState *>(sw);
    const int t = threadIdx.x;
    const unsigned long long *gw = reinterpret_cast<const unsigned long long *>(st);
    {
        // all of this thread's words in flight at once, then into LDS
        constexpr int SQ = (GSTATE_SMALL_WORDS + KT - 1) / KT;
        unsigned long long v[SQ];
#pragma unroll
        for (int q = 0; q < SQ; ++q) {
            const int k = t + q * KT;
            v[q] = k < GSTATE_SMALL_WORDS ? gw[k] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < SQ; ++q) {
            const int k = t + q * KT;
            if (k < GSTATE_SMALL_WORDS) sw[k] = v[q];
        }
    }
    double tot = strided_sum(part, nb);
    tot = block_sum(tot, red); // ends with a barrier: the staged state is complete
    if (ls->done) return;
    const int j = ls->j;
    double alpha, e, a2;
    const bool ok = reorth_scalars(ls, j, ls->hA, ls->hB, sc, &alpha, &e, &a2);
    // (tot is valid in thread 0 only)
    if (t < WAVE) dcgs_finish_wave(ls, st->H, MAXM, col, ok, alpha, e, a2, read_lane(tot, 0));
    __syncthreads();
    unsigned long long *gwo = reinterpret_cast<unsigned long long *>(st);
    for (int k = t; k < GSTATE_SMALL_WORDS; k += KT) gwo[k] = sw[k];
}

} // namespace gs2
