// Sliced-ELL copy of the system matrix for the Krylov solvers' SpMV.
#include <algorithm>
#include <vector>

#include "sella.hpp"

namespace gs2 {

// entries stored per slice: 64 * ceil(longest row of the slice / K); the
// element at index nslices is zero so that an exclusive scan ends the list
__global__ void k_sella_len(int64_t n, int64_t nslices, int K, const int32_t *__restrict__ rp,
                            int64_t *__restrict__ len)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s > nslices) return;
    if (s == nslices) {
        len[s] = 0;
        return;
    }
    const int C = WAVE / K;
    int m = 0;
    for (int r = 0; r < C; ++r) {
        const int64_t row = s * C + r;
        if (row < n) m = max(m, rp[row + 1] - rp[row]);
    }
    len[s] = (int64_t)WAVE * ((m + K - 1) / K);
}

// One thread per (slice, lane): lane l = r*K + q holds entries t*K + q of
// row r at step t; padding is (own column, 0).  Columns are written when
// with_col, else compared when flag is set (FILL_CHANGED).
__global__ void k_sella_fill(int64_t n, int64_t nslices, int K, const int32_t *__restrict__ rp,
                             const int32_t *__restrict__ ci, const double *__restrict__ va,
                             const int64_t *__restrict__ sp, int with_col, int32_t *__restrict__ col,
                             double *__restrict__ val, int *__restrict__ flag)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t s = gid / WAVE;
    if (s >= nslices) return;
    const int l = (int)(gid % WAVE), C = WAVE / K, r = l / K, q = l % K;
    const int64_t row = s * C + r;
    const int64_t beg = sp[s];
    const int steps = (int)((sp[s + 1] - beg) / WAVE);
    const int64_t b = row < n ? rp[row] : 0;
    const int len = row < n ? rp[row + 1] - rp[row] : 0;
    const int32_t pad = (int32_t)(row < n ? row : n - 1);
    bool changed = len > steps * K;
    for (int t = 0; t < steps; ++t) {
        const int e = t * K + q;
        const int64_t pos = beg + (int64_t)t * WAVE + l;
        const bool real = e < len;
        if (with_col) col[pos] = real ? ci[b + e] : pad;
        else if (flag && real && col[pos] != ci[b + e]) changed = true;
        val[pos] = real ? va[b + e] : 0.0;
    }
    if (flag && changed) atomicOr(flag, FILL_CHANGED);
}

void sella_free(SellA &S)
{
    for (void *p : {S.mem[0], S.mem[1]})
        if (p) (void)hipFree(p);
    S = SellA{};
}

struct DiaOffsA {
    int nd;
    int off[DIA_MAX];
};

// Values of the diagonal (B3 = false) or 3-row block (B3 = true) copy: entry
// (i, c) goes to diagonal t (the index of c - i among the offsets) at row i's
// position (interleaved by R rows per lane), or to plane
// 9 t + 3 (i mod 3) + (c mod 3) (t the index of the node offset c/3 - i/3)
// at node i/3's position.  A workgroup forms its tile, FILL_ROWS rows or
// FILL_NODES nodes of every plane, in LDS and writes it whole, absent entries
// as zeros, in stores of full 128-byte lines.  This runs at every solve (the
// values may have changed in place); bound by the copy's bytes.  Storing each
// entry on its own, 8 bytes to as many planes as a row has entries, took
// 1.46 ms per solve on the 64^3 elasticity matrix (27 node offsets), this 0.52.
// flag: FILL_CHANGED where an entry has no place in the layout,
// FILL_UNSORTED where a row's columns do not increase.
constexpr int FILL_ROWS = 128, FILL_NODES = 16, FILL_TB = 256;

template <bool B3>
__global__ __launch_bounds__(FILL_TB) void k_copy_fill(int64_t n, int R, const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ ci,
                                                       const double *__restrict__ va, DiaOffsA o, int64_t stride,
                                                       double *__restrict__ val, int *__restrict__ flag)
{
    constexpr int T = B3 ? FILL_NODES : FILL_ROWS, ROWS = B3 ? 3 * T : T, LANES = B3 ? 16 : 8;
    constexpr int LD = T + 1; // an odd leading dimension: a row's entries fall into different banks
    extern __shared__ double tile[];
    __shared__ int soff[DIA_MAX];
    if (threadIdx.x == 0) {
#pragma unroll
        for (int d = 0; d < DIA_MAX; ++d) soff[d] = o.off[d];
    }
    const int planes = B3 ? 9 * o.nd : o.nd;
    for (int k = threadIdx.x; k < planes * LD; k += FILL_TB) tile[k] = 0.0;
    __syncthreads();
    const int32_t i0 = (int32_t)blockIdx.x * ROWS;
    int bad = 0;
    for (int l = threadIdx.x / LANES; l < ROWS; l += FILL_TB / LANES) {
        const int32_t i = i0 + l;
        if (i >= n) break;
        int pos = l / 3;
        if constexpr (!B3) {
            const int blk = WAVE * R;
            pos = (l / blk) * blk + (l % WAVE) * R + (l % blk) / WAVE;
        }
        const int32_t b = rp[i], e = rp[i + 1], node = i / 3;
        for (int32_t k = b + (int32_t)(threadIdx.x % LANES); k < e; k += LANES) {
            const int32_t c = ci[k];
            if (k > b && ci[k - 1] >= c) bad |= FILL_UNSORTED;
            const int32_t d = B3 ? c / 3 - node : c - i;
            // where a row has an entry for every offset before c's, the
            // entry's number tells the offset's; else a binary search
            int lo = min(B3 ? (k - b) / 3 : k - b, o.nd - 1);
            if (soff[lo] != d) {
                int hi = o.nd - 1;
                lo = 0;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (soff[mid] < d) lo = mid + 1;
                    else hi = mid;
                }
            }
            if (soff[lo] != d) bad |= FILL_CHANGED;
            else tile[(B3 ? 9 * lo + 3 * (i - 3 * node) + (c - 3 * (c / 3)) : lo) * LD + pos] = va[k];
        }
    }
    if (flag && bad) atomicOr(flag, bad);
    __syncthreads();
    double *out = val + (int64_t)blockIdx.x * T;
    for (int k = threadIdx.x; k < planes * T; k += FILL_TB) out[(int64_t)(k / T) * stride + k % T] = tile[(k / T) * LD + k % T];
}

int sella_build_dia(SellA &S, const gs2_csr &A, int R, const std::vector<int> &offs, hipStream_t s)
{
    sella_free(S);
    S.n = A.n;
    S.nnz = A.nnz;
    S.dR = R;
    S.ndiag = (int)offs.size();
    S.dstride = std::max<int64_t>(1, (A.n + KRB - 1) / KRB) * KRB;
    for (int d = 0; d < DIA_MAX; ++d) S.doff[d] = d < S.ndiag ? offs[d] : 0;
    const size_t bytes = sizeof(double) * (size_t)std::max(S.ndiag, 1) * (size_t)S.dstride;
    GS2_TRY_HIP(hipMalloc(&S.mem[0], bytes));
    S.dval = (double *)S.mem[0];
    GS2_TRY_HIP(hipMemsetAsync(S.dval, 0, bytes, s));
    S.sel = -R;
    return GS2_OK;
}

int sella_build_b3(SellA &S, const gs2_csr &A, int R, const std::vector<int> &offs, hipStream_t s)
{
    sella_free(S);
    S.n = A.n;
    S.nnz = A.nnz;
    S.dR = R;
    S.ndiag = (int)offs.size();
    S.dstride = std::max<int64_t>(1, (A.n / 3 + KRB - 1) / KRB) * KRB; // nodes
    for (int d = 0; d < DIA_MAX; ++d) S.doff[d] = d < S.ndiag ? offs[d] : 0;
    const size_t bytes = sizeof(double) * 9 * (size_t)std::max(S.ndiag, 1) * (size_t)S.dstride;
    GS2_TRY_HIP(hipMalloc(&S.mem[0], bytes));
    S.dval = (double *)S.mem[0];
    GS2_TRY_HIP(hipMemsetAsync(S.dval, 0, bytes, s));
    S.sel = -10 - R;
    return GS2_OK;
}

// copy A's values into the built layout
int sella_fill_values(SellA &S, const gs2_csr &A, bool with_col, hipStream_t s, int *flag)
{
    const int tb = 256;
    if (S.sel < 0) {
        if (A.n > 0 && S.ndiag > 0) {
            DiaOffsA o;
            o.nd = S.ndiag;
            for (int d = 0; d < DIA_MAX; ++d) o.off[d] = S.doff[d];
            if (S.sel <= -10) {
                const unsigned g = (unsigned)((A.n / 3 + FILL_NODES - 1) / FILL_NODES);
                k_copy_fill<true><<<g, FILL_TB, sizeof(double) * 9 * o.nd * (FILL_NODES + 1), s>>>(
                    A.n, 1, A.rowptr, A.colind, A.val, o, S.dstride, S.dval, flag);
            } else {
                const unsigned g = (unsigned)((A.n + FILL_ROWS - 1) / FILL_ROWS);
                k_copy_fill<false><<<g, FILL_TB, sizeof(double) * o.nd * (FILL_ROWS + 1), s>>>(
                    A.n, S.dR, A.rowptr, A.colind, A.val, o, S.dstride, S.dval, flag);
            }
        }
    } else if (S.nslices > 0) {
        const int64_t threads = S.nslices * WAVE;
        k_sella_fill<<<(unsigned)((threads + tb - 1) / tb), tb, 0, s>>>(A.n, S.nslices, S.K, A.rowptr, A.colind,
                                                                       A.val, S.sp, with_col ? 1 : 0, S.col, S.val,
                                                                       flag);
    }
    GS2_TRY_HIP(hipGetLastError());
    return GS2_OK;
}

// Lanes per row: from K0 (the rule: the mean row length, as for the
// triangles), K grows while a few long rows would pad the copy beyond twice
// the entries.
static int sella_structure(SellA &S, const gs2_csr &A, int K0, hipStream_t s)
{
    const int tb = 256;
    for (int K = K0;; K *= 2) {
        S.K = K;
        S.C = WAVE / K;
        S.nslices = (A.n + S.C - 1) / S.C;
        const int64_t m = S.nslices + 1;
        // pointers, lengths, scan totals
        if (S.mem[0]) GS2_TRY_HIP(hipFree(S.mem[0]));
        S.mem[0] = nullptr;
        GS2_TRY_HIP(hipMalloc(&S.mem[0], sizeof(int64_t) * (2 * m + scan_tmp(m))));
        S.sp = (int64_t *)S.mem[0];
        k_sella_len<<<(unsigned)((m + tb - 1) / tb), tb, 0, s>>>(A.n, S.nslices, K, A.rowptr, S.sp + m);
        GS2_TRY(exclusive_scan_i64(S.sp + m, S.sp, m, S.sp + 2 * m, s));
        GS2_TRY_HIP(hipMemcpyAsync(&S.padded, S.sp + S.nslices, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        GS2_TRY_HIP(hipStreamSynchronize(s));
        if (K == WAVE || S.padded <= 2 * A.nnz + WAVE * S.nslices) break;
    }
    const size_t cnt = (size_t)std::max<int64_t>(S.padded, WAVE), vb = aligned(sizeof(double) * cnt);
    GS2_TRY_HIP(hipMalloc(&S.mem[1], vb + sizeof(int32_t) * cnt));
    S.val = (double *)S.mem[1];
    S.col = (int32_t *)((char *)S.mem[1] + vb);
    return GS2_OK;
}

int sella_rule_lanes(const gs2_csr &A) { return choose_lanes((double)A.nnz / (double)std::max<int64_t>(A.n, 1), 0); }

// Sliced-ELL structure with at least K0 lanes per row (columns and values
// filled), replacing whatever S held.
int sella_build_sell(SellA &S, const gs2_csr &A, int K0, hipStream_t s)
{
    sella_free(S);
    S.n = A.n;
    S.nnz = A.nnz;
    int st = sella_structure(S, A, K0, s);
    if (st == GS2_OK) {
        S.sel = S.K;
        st = sella_fill_values(S, A, true, s);
    }
    if (st != GS2_OK) sella_free(S);
    return st;
}

// The offsets for a copy without column indices; the stored values (padding
// included) may be at most 1.5 times the entries.
bool sella_dia_offsets(const gs2_csr &A, const Pattern &P, std::vector<int> &offs)
{
    if (P.many_d || A.n <= 0 || A.n > (int64_t(1) << 30) || (int)P.d.size() > DIA_MAX) return false;
    offs = P.d;
    return (double)offs.size() * (double)A.n <= 1.5 * (double)A.nnz + (double)KRB * offs.size();
}

bool sella_b3_offsets(const gs2_csr &A, const Pattern &P, std::vector<int> &offs)
{
    if (P.many_b || A.n <= 0 || A.n > (int64_t(1) << 30)) return false;
    offs = P.bl;
    offs.insert(offs.end(), P.bu.begin(), P.bu.end());
    if (std::binary_search(P.d.begin(), P.d.end(), 0) || P.many_d) offs.push_back(0); // a diagonal entry
    std::sort(offs.begin(), offs.end());
    offs.erase(std::unique(offs.begin(), offs.end()), offs.end());
    return (int)offs.size() <= DIA_MAX &&
           3.0 * (double)offs.size() * (double)A.n <= 1.5 * (double)A.nnz + 3.0 * (double)KRB * offs.size();
}

} // namespace gs2
