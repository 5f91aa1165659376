// GS2 setup (Sections 3 and 6): validate the CSR input, extract D, build the
// scaling vectors, split the scaled matrix into its strictly lower and upper
// triangles in sliced-ELL layout and the requested precision, optionally
// build level sets, and pick a lane-per-row schedule.  The paper notes that
// GS2 needs no eigenvalue estimate and only this cheap setup (Section 12).

#include <algorithm>
#include <chrono>
#include <cmath>
#include <new>

#include "gs2_internal.hpp"

namespace gs2 {

enum : int { ERRF_BAD_CSR = 1, ERRF_ZERO_DIAG = 2, ERRF_NONFINITE = 4, ERRF_FP16 = 8 };

static int flags_to_status(int f)
{
    if (f & ERRF_BAD_CSR) return GS2_ERR_BAD_CSR;
    if (f & ERRF_ZERO_DIAG) return GS2_ERR_ZERO_DIAG;
    if (f & ERRF_NONFINITE) return GS2_ERR_NONFINITE;
    if (f & ERRF_FP16) return GS2_ERR_FP16_RANGE;
    return GS2_OK;
}

// ------------------------------------------------------- pattern scan
//
// One pass over the CSR input: structural checks, triangle counts, scaling
// vectors, and the distinct offsets that decide whether the diagonal or the
// 3-row block layout fits.  LN threads per row take every LN-th entry.  The
// distinct offsets collect in hash tables in LDS (a stencil's entries find
// theirs on the first probe), which every workgroup folds into the device's
// at its end; a table that meets more keys than two triangles could have is
// given up.  64^3 elasticity (61 M entries): 0.50 ms, where the checks alone
// with one thread per row took 2.0 ms and the offsets a copy of the pattern
// and a loop on the host.  90 x 84 x 77 diffusion (4 M entries): 0.11 ms.
constexpr int PT_SLOTS = 128, PT_MOST = 2 * DIA_MAX + 1, PT_EMPTY = INT32_MIN, PT_FAR = 1024;

struct PatternDev {
    int err, maxlen, lo, hi, many_d, many_b;
    unsigned long long nl, nu, far;
    int d[PT_SLOTS], bl[PT_SLOTS], bu[PT_SLOTS];
};
size_t pattern_dev_bytes() { return aligned(sizeof(PatternDev)); }

__global__ void k_pattern_init(PatternDev *st)
{
    const int t = threadIdx.x;
    if (t < PT_SLOTS) st->d[t] = st->bl[t] = st->bu[t] = PT_EMPTY;
    if (t == 0) {
        st->err = st->maxlen = st->lo = st->hi = st->many_d = st->many_b = 0;
        st->nl = st->nu = st->far = 0;
    }
}

// false when the table has no room for the key
__device__ __forceinline__ bool table_add(int *keys, int key)
{
    unsigned h = (unsigned)key * 2654435761u >> 25;
    for (int p = 0; p < PT_SLOTS; ++p) {
        const int k = keys[h];
        if (k == key) return true;
        if (k == PT_EMPTY) {
            const int old = atomicCAS(&keys[h], PT_EMPTY, key);
            if (old == PT_EMPTY || old == key) return true;
        }
        h = (h + 1) % PT_SLOTS;
    }
    return false;
}

template <int LN, bool VALUES>
__global__ __launch_bounds__(256) void k_scan_pattern(int64_t n, int64_t nnz, const int32_t *__restrict__ rp,
                                                      const int32_t *__restrict__ ci, const double *__restrict__ va,
                                                      int32_t *__restrict__ lcnt, int32_t *__restrict__ ucnt,
                                                      double *__restrict__ sl, double *__restrict__ sr,
                                                      PatternDev *st)
{
    __shared__ int td[PT_SLOTS], tl[PT_SLOTS], tu[PT_SLOTS], many[2], sums[4];
    __shared__ unsigned long long cnt[3];
    const int t = threadIdx.x, q = t % LN;
    for (int k = t; k < PT_SLOTS; k += 256) td[k] = tl[k] = tu[k] = PT_EMPTY;
    if (t == 0) {
        many[0] = st->many_d;
        many[1] = n % 3 != 0 || st->many_b;
        sums[0] = sums[1] = sums[2] = sums[3] = 0;
        cnt[0] = cnt[1] = cnt[2] = 0;
    }
    __syncthreads();
    int f = 0, longest = 0, lo = 0, hi = 0;
    unsigned long long nls = 0, nus = 0, far = 0;
    if (blockIdx.x == 0 && t == 0 && (rp[0] != 0 || rp[n] != nnz)) f |= ERRF_BAD_CSR;
    const int64_t step = (int64_t)gridDim.x * (256 / LN);
    for (int64_t i = (int64_t)blockIdx.x * (256 / LN) + t / LN; i < n; i += step) {
        const int64_t b = rp[i], e = rp[i + 1];
        if (b < 0 || e < b || e > nnz) {
            f |= ERRF_BAD_CSR;
            continue;
        }
        int nl = 0, nu = 0, found = 0;
        double dv = 0.0;
        const int node = (int)i / 3;
        for (int64_t k = b + q; k < e; k += LN) {
            const int c = ci[k];
            const bool bad = c <= (k > b ? ci[k - 1] : -1) || c >= n;
            double v = 0.0;
            if constexpr (VALUES) {
                v = va[k];
                if (!isfinite(v)) f |= ERRF_NONFINITE;
            }
            if (c < i) ++nl;
            else if (c > i) ++nu;
            else {
                found = 1;
                dv = v;
            }
            if (bad) {
                f |= ERRF_BAD_CSR;
                continue;
            }
            const int d = (int)(c - i);
            lo = min(lo, d);
            hi = max(hi, d);
            far += abs(d) > PT_FAR;
            if (!many[0] && !table_add(td, d)) many[0] = 1;
            if (!many[1] && d != 0 && !table_add(d < 0 ? tl : tu, c / 3 - node)) many[1] = 1;
        }
#pragma unroll
        for (int o = 1; o < LN; o <<= 1) {
            nl += __shfl_xor(nl, o);
            nu += __shfl_xor(nu, o);
            found |= __shfl_xor(found, o);
            dv += __shfl_xor(dv, o);
        }
        if (q == 0) {
            nls += nl;
            nus += nu;
            longest = max(longest, (int)(e - b) - 1);
            if constexpr (VALUES) {
                if (!found || dv == 0.0) f |= ERRF_ZERO_DIAG;
                lcnt[i] = nl;
                ucnt[i] = nu;
                const double sc = 1.0 / sqrt(fabs(dv));
                sr[i] = sc;
                sl[i] = dv < 0.0 ? -sc : sc;
            }
        }
    }
    if (f) atomicOr(&sums[0], f);
    if (longest) atomicMax(&sums[1], longest);
    if (lo) atomicMin(&sums[2], lo);
    if (hi) atomicMax(&sums[3], hi);
    if (nls) atomicAdd(&cnt[0], nls);
    if (nus) atomicAdd(&cnt[1], nus);
    if (far) atomicAdd(&cnt[2], far);
    __syncthreads();
    if (t == 0) {
        if (sums[0]) atomicOr(&st->err, sums[0]);
        // a plain read first: after a few workgroups the extremes stand
        if (sums[1] > st->maxlen) atomicMax(&st->maxlen, sums[1]);
        if (sums[2] < st->lo) atomicMin(&st->lo, sums[2]);
        if (sums[3] > st->hi) atomicMax(&st->hi, sums[3]);
        atomicAdd(&st->nl, cnt[0]);
        atomicAdd(&st->nu, cnt[1]);
        if (cnt[2]) atomicAdd(&st->far, cnt[2]);
    }
    // the keys into the device's tables (found by a plain read after the first workgroups)
    if (t < PT_SLOTS) {
        if (td[t] != PT_EMPTY && !many[0] && !table_add(st->d, td[t])) many[0] = 1;
        if (!many[1] && tl[t] != PT_EMPTY && !table_add(st->bl, tl[t])) many[1] = 1;
        if (!many[1] && tu[t] != PT_EMPTY && !table_add(st->bu, tu[t])) many[1] = 1;
    }
    __syncthreads();
    if (t == 0) {
        if (many[0]) st->many_d = 1;
        if (many[1]) st->many_b = 1;
    }
}

static void table_list(const int *keys, std::vector<int> &out, bool &many)
{
    for (int k = 0; k < PT_SLOTS; ++k)
        if (keys[k] != PT_EMPTY) out.push_back(keys[k]);
    std::sort(out.begin(), out.end());
    many = many || (int)out.size() > PT_MOST;
}

int scan_pattern(const gs2_csr &A, int32_t *lcnt, int32_t *ucnt, double *sl, double *sr, PatternDev *dev, Pattern &out,
                 hipStream_t s)
{
    out = Pattern{};
    k_pattern_init<<<1, PT_SLOTS, 0, s>>>(dev);
    // 8 threads per row for stencil rows, 32 for long ones; 16 groups of rows
    // and more per workgroup, 2048 workgroups at most, so that folding the
    // tables and counts, one workgroup after the other, stays small
    const bool wide = A.nnz > 24 * A.n;
    const int per = 256 / (wide ? 32 : 8);
    const int64_t groups = (A.n + per - 1) / per;
    const unsigned g = (unsigned)std::min<int64_t>(groups, std::min<int64_t>(std::max<int64_t>(256, groups / 16), 2048));
    if (lcnt) {
        if (wide) k_scan_pattern<32, true><<<g, 256, 0, s>>>(A.n, A.nnz, A.rowptr, A.colind, A.val, lcnt, ucnt, sl, sr, dev);
        else k_scan_pattern<8, true><<<g, 256, 0, s>>>(A.n, A.nnz, A.rowptr, A.colind, A.val, lcnt, ucnt, sl, sr, dev);
    } else {
        if (wide) k_scan_pattern<32, false><<<g, 256, 0, s>>>(A.n, A.nnz, A.rowptr, A.colind, nullptr, nullptr, nullptr, nullptr, nullptr, dev);
        else k_scan_pattern<8, false><<<g, 256, 0, s>>>(A.n, A.nnz, A.rowptr, A.colind, nullptr, nullptr, nullptr, nullptr, nullptr, dev);
    }
    GS2_TRY_HIP(hipGetLastError());
    PatternDev h;
    GS2_TRY_HIP(hipMemcpyAsync(&h, dev, sizeof(h), hipMemcpyDeviceToHost, s));
    GS2_TRY_HIP(hipStreamSynchronize(s));
    out.err = h.err;
    out.maxlen = h.maxlen;
    out.lo = h.lo;
    out.hi = h.hi;
    out.nl = (int64_t)h.nl;
    out.nu = (int64_t)h.nu;
    out.far = (int64_t)h.far;
    out.many_d = h.many_d != 0;
    out.many_b = A.n % 3 != 0 || h.many_b != 0;
    table_list(h.d, out.d, out.many_d);
    table_list(h.bl, out.bl, out.many_b);
    table_list(h.bu, out.bu, out.many_b);
    return GS2_OK;
}

// IEEE binary16 round-to-nearest-even of a float64, by integer manipulation of
// the binary64 encoding.  Returns the 16-bit pattern; sets *ovf if the
// result is infinite or NaN.
__device__ __forceinline__ uint16_t f64_to_f16_bits(double x, int *ovf)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
    const int ex = (int)((b >> 52) & 0x7ff);
    const uint64_t man = b & ((1ull << 52) - 1);
    if (ex == 0x7ff) { *ovf = 1; return sign | 0x7e00u; }
    if (ex == 0) return sign; // binary64 zero / subnormal: far below half's range
    const int e = ex - 1023;
    if (e > 15) { *ovf = 1; return sign | 0x7c00u; }
    const int E = e < -14 ? -14 : e;
    const int shift = 42 + (E - e); // bits of the 53-bit significand below half's quantum
    if (shift >= 54) return sign;
    const uint64_t m = man | (1ull << 52);
    uint64_t N = m >> shift;
    const uint64_t rem = m & ((1ull << shift) - 1), halfq = 1ull << (shift - 1);
    if (rem > halfq || (rem == halfq && (N & 1))) ++N;
    const uint32_t bits = ((uint32_t)(E + 14) << 10) + (uint32_t)N;
    if (bits >= 0x7c00u) { *ovf = 1; return sign | 0x7c00u; }
    return sign | (uint16_t)bits;
}

template <typename VT>
__device__ __forceinline__ VT convert_scaled(double v, int *ovf);
template <>
__device__ __forceinline__ double convert_scaled<double>(double v, int *) { return v; }
template <>
__device__ __forceinline__ float convert_scaled<float>(double v, int *ovf)
{
    const float f = (float)v;
    if (!isfinite(f)) *ovf = 1;
    return f;
}
template <>
__device__ __forceinline__ _Float16 convert_scaled<_Float16>(double v, int *ovf)
{
    const uint16_t bits = f64_to_f16_bits(v, ovf);
    _Float16 h;
    __builtin_memcpy(&h, &bits, 2);
    return h;
}

// Which entries of a row a stored part holds, as up to two ranges of the
// row's sorted CSR entries.  Parts: 0 = strictly lower inside the row's
// block, 1 = strictly upper inside the block, 2 = outside the block (the
// couplings of the hybrid relaxation).  Blocks are contiguous ranges of bs
// rows; with one block (bs >= n) part 2 is empty.  Sorted columns put the
// off-block lower entries first and the off-block upper entries last.
enum : int { PART_L = 0, PART_U = 1, PART_E = 2 };

struct Rows {
    const int32_t *rp, *ci, *lcnt, *ucnt;
    int64_t n, bs;
};

struct Range {
    int o1, c1, o2, c2;
};

__device__ __forceinline__ Range row_range(const Rows &A, int part, int64_t i)
{
    const int lc = A.lcnt[i], uc = A.ucnt[i];
    int lo = 0, hi = 0;
    if (A.bs < A.n) {
        const int64_t b0 = (i / A.bs) * A.bs, b1 = b0 + A.bs < A.n ? b0 + A.bs : A.n, r = A.rp[i];
        while (lo < lc && A.ci[r + lo] < b0) ++lo;
        while (hi < uc && A.ci[r + lc + uc - hi] >= b1) ++hi;
    }
    if (part == PART_L) return Range{lo, lc - lo, 0, 0};
    if (part == PART_U) return Range{lc + 1, uc - hi, 0, 0};
    return Range{0, lo, lc + 1 + uc - hi, hi};
}

// Stored entries of each slice of a part: 64 * ceil(longest row / K), one
// lane per row.  The extra element at index nslices is zero so that an
// exclusive scan yields the end.  With st, adds up the part's entries and their
// smallest and largest col - row (one workgroup after the other: only where what
// the pattern scan found does not hold, with several blocks).
struct PartStats {
    unsigned long long total;
    int lo, hi; // 0 among them, as padding
};
__global__ __launch_bounds__(256) void k_slice_len(Rows A, int part, int64_t nslices, int K, int64_t *__restrict__ len,
                                                   PartStats *st)
{
    const int C = WAVE / K;
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int c = 0, lo = 0, hi = 0;
    if (row < A.n) {
        const Range r = row_range(A, part, row);
        c = r.c1 + r.c2;
        if (st && c > 0) {
            const int64_t b = A.rp[row];
            lo = min(0, A.ci[b + (r.c1 ? r.o1 : r.o2)] - (int)row);
            hi = max(0, A.ci[b + (r.c2 ? r.o2 + r.c2 : r.o1 + r.c1) - 1] - (int)row);
        }
    }
    int m = c;
    for (int o = 1; o < C; o <<= 1) m = max(m, __shfl_xor(m, o));
    if (st) {
        __shared__ int sum, los, his;
        if (threadIdx.x == 0) sum = los = his = 0;
        __syncthreads();
        int t = c;
        for (int o = 1; o < WAVE; o <<= 1) {
            t += __shfl_xor(t, o);
            lo = min(lo, __shfl_xor(lo, o));
            hi = max(hi, __shfl_xor(hi, o));
        }
        if (threadIdx.x % WAVE == 0 && t) {
            atomicAdd(&sum, t);
            atomicMin(&los, lo);
            atomicMax(&his, hi);
        }
        __syncthreads();
        if (threadIdx.x == 0 && sum) {
            atomicAdd(&st->total, (unsigned long long)sum);
            // a plain read first: after a few workgroups the extremes stand
            if (los < st->lo) atomicMin(&st->lo, los);
            if (his > st->hi) atomicMax(&st->hi, his);
        }
    }
    if (row % C == 0 && row / C <= nslices) len[row / C] = row / C == nslices ? 0 : (int64_t)WAVE * ((m + K - 1) / K);
}

// One thread per (slice, lane): writes the lane's entries of its row, the
// value (s_l[i] * a_ij) * s_r[j] rounded once to VT, padding with
// (own column, 0); with off, the columns' 16-bit form col - row - off_min too.
template <typename VT>
__global__ void k_fill(Rows A, int part, int64_t nslices, int K, const double *__restrict__ va,
                       const double *__restrict__ sl, const double *__restrict__ sr, const int64_t *__restrict__ sp,
                       int32_t *__restrict__ col, uint16_t *__restrict__ off, int off_min, VT *__restrict__ val,
                       int *__restrict__ err)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t s = gid / WAVE;
    if (s >= nslices) return;
    const int l = (int)(gid % WAVE);
    const int C = WAVE / K;
    const int r = l / K, q = l % K;
    const int64_t row = s * C + r, n = A.n;
    const int64_t beg = sp[s];
    const int steps = (int)((sp[s + 1] - beg) / WAVE);
    const Range rg = row < n ? row_range(A, part, row) : Range{0, 0, 0, 0};
    const int64_t base = row < n ? (int64_t)A.rp[row] : 0;
    const int32_t pad_col = (int32_t)(row < n ? row : n - 1);
    const double srow = row < n ? sl[row] : 0.0;
    int ovf = 0;
    for (int t = 0; t < steps; ++t) {
        const int e = t * K + q;
        const int64_t pos = beg + (int64_t)t * WAVE + l;
        int32_t c = pad_col;
        VT v = VT(0);
        if (e < rg.c1 + rg.c2) {
            const int64_t idx = base + (e < rg.c1 ? rg.o1 + e : rg.o2 + (e - rg.c1));
            c = A.ci[idx];
            v = convert_scaled<VT>((srow * va[idx]) * sr[c], &ovf);
        }
        col[pos] = c;
        val[pos] = v;
        if (off) off[pos] = (uint16_t)(c - (int)row - off_min);
    }
    if (ovf) atomicOr(err, ERRF_FP16);
}

void free_sell(Sell &S)
{
    for (void *&p : S.mem) {
        if (p) (void)hipFree(p);
        p = nullptr;
    }
    S.slice_ptr = nullptr;
    S.col = nullptr;
    S.off = nullptr;
    S.val = nullptr;
}

// ------------------------------------------- diagonal-interleaved triangles

void free_dia(Dia &D)
{
    if (D.mem) (void)hipFree(D.mem);
    D.mem = D.val = nullptr;
}

struct DiaOffs {
    int nd;
    int off[DIA_MAX];
};

// One thread per row: the row's entries of one part go to their diagonal at
// the row's interleaved position, value (s_l[i] * a_ij) * s_r[j] rounded once
// to VT.  The array is zeroed beforehand (rows past n and absent entries).
template <typename VT>
__global__ void k_dia_fill(int64_t n, int R, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                           const double *__restrict__ va, const int32_t *__restrict__ lcnt, int lower, DiaOffs o,
                           const double *__restrict__ sl, const double *__restrict__ sr, int64_t stride,
                           VT *__restrict__ val, int *__restrict__ err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t blk = (int64_t)WAVE * R;
    const int64_t pos = (i / blk) * blk + (i % WAVE) * R + (i % blk) / WAVE;
    const int64_t b = lower ? rp[i] : rp[i] + lcnt[i] + 1, e = lower ? rp[i] + lcnt[i] : rp[i + 1];
    const double srow = sl[i];
    int t = 0, ovf = 0;
    for (int64_t k = b; k < e; ++k) {
        const int c = ci[k];
        const int d = (int)((int64_t)c - i);
        while (t < o.nd - 1 && o.off[t] < d) ++t; // offsets ascend within a row
        if (o.off[t] != d) {
            atomicOr(err, ERRF_BAD_CSR); // cannot happen for a pattern the offsets came from
            return;
        }
        val[(int64_t)t * stride + pos] = convert_scaled<VT>((srow * va[k]) * sr[c], &ovf);
    }
    if (ovf) atomicOr(err, ERRF_FP16);
}

// The 3-row block layout: entry (i, c) of the part goes to plane
// 9 t + 3 (i mod 3) + (c mod 3), t the index of its node offset c/3 - i/3,
// at node i/3's interleaved position (R nodes per lane); scaled and rounded
// as in k_dia_fill.
template <typename VT>
__global__ void k_b3_fill(int64_t n, int R, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                          const double *__restrict__ va, const int32_t *__restrict__ lcnt, int lower, DiaOffs o,
                          const double *__restrict__ sl, const double *__restrict__ sr, int64_t stride,
                          VT *__restrict__ val, int *__restrict__ err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t blk = (int64_t)WAVE * R, node = i / 3, j = i - 3 * node;
    const int64_t pos = (node / blk) * blk + (node % WAVE) * R + (node % blk) / WAVE;
    const int64_t b = lower ? rp[i] : rp[i] + lcnt[i] + 1, e = lower ? rp[i] + lcnt[i] : rp[i + 1];
    const double srow = sl[i];
    int t = 0, ovf = 0;
    for (int64_t k = b; k < e; ++k) {
        const int c = ci[k];
        const int cn = c / 3;
        const int d = (int)((int64_t)cn - node);
        while (t < o.nd - 1 && o.off[t] < d) ++t; // node offsets ascend within a row
        if (o.off[t] != d) {
            atomicOr(err, ERRF_BAD_CSR); // cannot happen for a pattern the offsets came from
            return;
        }
        val[(int64_t)(9 * t + 3 * j + (c - 3 * cn)) * stride + pos] = convert_scaled<VT>((srow * va[k]) * sr[c], &ovf);
    }
    if (ovf) atomicOr(err, ERRF_FP16);
}

// Describe one triangle in the diagonal-interleaved layout with R rows per
// lane, or in the 3-row block layout with R nodes per lane; rows (nodes) are
// padded to whole workgroups of the sweep kernels (DIA_THREADS * R of them)
// so that every launched lane has a slot.  Returns its bytes.
static size_t shape_dia(Dia &D, int64_t n, int precision, int R, const std::vector<int> &offs, int64_t nnz, int b3)
{
    D.ndiag = (int)offs.size();
    D.R = R;
    D.nnz = nnz;
    D.b3 = b3;
    D.val_bytes = precision == GS2_FP64 ? 8 : precision == GS2_FP32 ? 4 : 2;
    const int64_t wg = (int64_t)DIA_THREADS * R, units = b3 ? n / 3 : n;
    D.stride = std::max<int64_t>(1, (units + wg - 1) / wg) * wg;
    for (int d = 0; d < DIA_MAX; ++d) D.off[d] = d < D.ndiag ? offs[d] : 0;
    return aligned((size_t)std::max(1, D.ndiag) * (b3 ? 9 : 1) * (size_t)D.stride * D.val_bytes);
}

template <typename VT>
static void fill_dia(const Dia &D, int64_t n, int lower, const gs2_csr &A, const int32_t *lcnt, const double *sl,
                     const double *sr, int *err, hipStream_t s)
{
    if (D.ndiag == 0 || n == 0) return;
    DiaOffs o;
    o.nd = D.ndiag;
    for (int d = 0; d < DIA_MAX; ++d) o.off[d] = D.off[d];
    const unsigned g = (unsigned)((n + 255) / 256);
    if (D.b3)
        k_b3_fill<VT><<<g, 256, 0, s>>>(n, D.R, A.rowptr, A.colind, A.val, lcnt, lower, o, sl, sr, D.stride, (VT *)D.val,
                                        err);
    else
        k_dia_fill<VT><<<g, 256, 0, s>>>(n, D.R, A.rowptr, A.colind, A.val, lcnt, lower, o, sl, sr, D.stride,
                                         (VT *)D.val, err);
}

// ------------------------------------------------------- exclusive scan
//
// out[i] = sum of in[0..i), for the slice pointers of the sliced-ELL arrays.
// Three passes: each workgroup scans its 1024 elements (four per thread, the
// thread totals combined by a Hillis-Steele scan in LDS) and writes its
// total; one workgroup scans the totals in chunks of 256 with a running
// carry; every element then adds its workgroup's offset.  Integer sums, so
// the result is exact whatever the order.
constexpr int SCAN_TB = 256, SCAN_PER = 4, SCAN_BLOCK = SCAN_TB * SCAN_PER;

__device__ __forceinline__ int64_t block_incl_scan(int64_t v, int64_t *sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < SCAN_TB; off <<= 1) {
        const int64_t x = t >= off ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    return sh[t];
}

__global__ __launch_bounds__(SCAN_TB) void k_scan_local(const int64_t *__restrict__ in, int64_t *__restrict__ out,
                                                        int64_t m, int64_t *__restrict__ bsum)
{
    __shared__ int64_t sh[SCAN_TB];
    const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + (int64_t)threadIdx.x * SCAN_PER;
    int64_t v[SCAN_PER], run = 0;
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q) {
        v[q] = base + q < m ? in[base + q] : 0;
        run += v[q];
    }
    const int64_t incl = block_incl_scan(run, sh);
    int64_t e = incl - run;
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q) {
        if (base + q < m) out[base + q] = e;
        e += v[q];
    }
    if (threadIdx.x == SCAN_TB - 1) bsum[blockIdx.x] = incl;
}

__global__ __launch_bounds__(SCAN_TB) void k_scan_sums(int64_t *__restrict__ bsum, int64_t nb)
{
    __shared__ int64_t sh[SCAN_TB];
    int64_t carry = 0; // the same in every thread
    for (int64_t c0 = 0; c0 < nb; c0 += SCAN_TB) {
        const int64_t i = c0 + threadIdx.x;
        const int64_t v = i < nb ? bsum[i] : 0;
        const int64_t incl = block_incl_scan(v, sh);
        if (i < nb) bsum[i] = carry + incl - v;
        carry += sh[SCAN_TB - 1];
        __syncthreads();
    }
}

__global__ __launch_bounds__(SCAN_TB) void k_scan_add(int64_t *__restrict__ out, int64_t m,
                                                      const int64_t *__restrict__ bsum)
{
    const int64_t i = (int64_t)blockIdx.x * SCAN_TB + threadIdx.x;
    if (i < m) out[i] += bsum[i / SCAN_BLOCK];
}

int64_t scan_tmp(int64_t m) { return (m + SCAN_BLOCK - 1) / SCAN_BLOCK; }

int exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t m, int64_t *tmp, hipStream_t s)
{
    if (m <= 0) return GS2_OK;
    const int64_t nb = scan_tmp(m);
    k_scan_local<<<(unsigned)nb, SCAN_TB, 0, s>>>(in, out, m, tmp);
    k_scan_sums<<<1, SCAN_TB, 0, s>>>(tmp, nb);
    k_scan_add<<<(unsigned)((m + SCAN_TB - 1) / SCAN_TB), SCAN_TB, 0, s>>>(out, m, tmp);
    GS2_TRY_HIP(hipGetLastError());
    return GS2_OK;
}

int choose_lanes(double avg_len, int max_len)
{
    (void)max_len;
    if (avg_len <= 12.0) return 1;
    if (avg_len <= 24.0) return 2;
    if (avg_len <= 48.0) return 4;
    if (avg_len <= 96.0) return 8;
    return 16;
}

// Timed choices, process-wide.  The sweep schedules are keyed by the size bucket,
// rounded mean row length, longest-row bucket, precision and what else they depend
// on; the solver's (layout of A, basis passes) by the exact sizes, as nothing shows
// that a timing holds for twice the rows.  Past CHOICES_MOST of them the table starts
// anew.
constexpr size_t CHOICES_MOST = 4096;
static std::mutex g_choice_mu;
static std::map<std::string, int> g_choices;

bool choice_get(const std::string &key, int *choice)
{
    std::lock_guard<std::mutex> lk(g_choice_mu);
    auto it = g_choices.find(key);
    if (it == g_choices.end()) return false;
    *choice = it->second;
    return true;
}

void choice_put(const std::string &key, int choice)
{
    std::lock_guard<std::mutex> lk(g_choice_mu);
    if (g_choices.size() >= CHOICES_MOST) g_choices.clear();
    g_choices[key] = choice;
}

std::string shape_key(int64_t n, double avg, int maxlen, int prec)
{
    int nb = 0;
    while ((int64_t(1) << nb) < n) ++nb;
    int mb = 0;
    while ((1 << mb) < maxlen) ++mb;
    char buf[96];
    std::snprintf(buf, sizeof buf, "n%d_a%d_m%d_p%d", nb, (int)std::lround(avg), mb, prec);
    return buf;
}

std::string size_key(int64_t n, int64_t m, int maxlen)
{
    return "n" + std::to_string(n) + "_" + std::to_string(m) + "_m" + std::to_string(maxlen);
}

// Device scratch of one setup, in one allocation.
struct SetupScratch {
    void *mem = nullptr;
    int32_t *lcnt = nullptr, *ucnt = nullptr;
    int *err = nullptr;
    PatternDev *dev = nullptr;
    Pattern pat;
    int alloc(int64_t n)
    {
        const size_t cnt = aligned(sizeof(int32_t) * n);
        GS2_TRY_HIP(hipMalloc(&mem, 2 * cnt + pattern_dev_bytes() + aligned(sizeof(int))));
        char *p = (char *)mem;
        lcnt = (int32_t *)p;
        ucnt = (int32_t *)(p + cnt);
        dev = (PatternDev *)(p + 2 * cnt);
        err = (int *)(p + 2 * cnt + pattern_dev_bytes());
        return GS2_OK;
    }
    ~SetupScratch()
    {
        if (mem) (void)hipFree(mem);
    }
};

template <typename VT>
static void fill_part(const Handle &h, const Sell &S, int part, const Rows &R, const gs2_csr &A, int *err, hipStream_t s)
{
    k_fill<VT><<<(unsigned)((S.nslices * WAVE + 255) / 256), 256, 0, s>>>(R, part, S.nslices, S.K, A.val, h.sl, h.sr,
                                                                         S.slice_ptr, S.col, S.off, S.off_min,
                                                                         (VT *)S.val, err);
}

// The parts [first, last] in sliced-ELL with K lanes per row, their slice
// pointers in one allocation and their entries in another, both owned by the
// first.  16-bit column offsets where the pattern's span allows them.
static int build_parts(Handle &h, int first, int last, int K, const gs2_csr &A, const SetupScratch &sc, hipStream_t s)
{
    Sell *const part[3] = {&h.L, &h.U, &h.E};
    const int np = last - first + 1;
    const int64_t n = h.n;
    const Rows R{A.rowptr, A.colind, sc.lcnt, sc.ucnt, n, h.blocks > 1 ? (n + h.blocks - 1) / h.blocks : n};
    const int vb = h.precision == GS2_FP64 ? 8 : h.precision == GS2_FP32 ? 4 : 2;
    const int64_t C = WAVE / K, ns = (n + C - 1) / C, tmp = scan_tmp(ns + 1);
    for (int q = first; q <= last; ++q) free_sell(*part[q]);
    Sell &own = *part[first];
    // per part: pointers, lengths, scan totals, counts
    const int64_t per = 2 * (ns + 1) + tmp + (int64_t)(sizeof(PartStats) / sizeof(int64_t));
    GS2_TRY_HIP(hipMalloc(&own.mem[0], sizeof(int64_t) * per * np));
    int64_t *base = (int64_t *)own.mem[0];
    int64_t ends[3];
    PartStats stats[3];
    for (int q = 0; q < np; ++q) {
        Sell &S = *part[first + q];
        S.n = n;
        S.K = K;
        S.C = (int)C;
        S.nslices = ns;
        S.val_bytes = vb;
        S.slice_ptr = base + q * per;
        int64_t *len = S.slice_ptr + ns + 1;
        PartStats *dev = (PartStats *)(len + ns + 1 + tmp);
        const bool count = h.blocks > 1;
        if (count) GS2_TRY_HIP(hipMemsetAsync(dev, 0, sizeof(PartStats), s));
        k_slice_len<<<(unsigned)((ns * C + 1 + 255) / 256), 256, 0, s>>>(R, first + q, ns, K, len, count ? dev : nullptr);
        GS2_TRY(exclusive_scan_i64(len, S.slice_ptr, ns + 1, len + ns + 1, s));
        GS2_TRY_HIP(hipMemcpyAsync(&ends[q], S.slice_ptr + ns, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        const bool low = first + q == PART_L;
        stats[q] = PartStats{(unsigned long long)(low ? sc.pat.nl : sc.pat.nu), low ? sc.pat.lo : 0, low ? 0 : sc.pat.hi};
        if (count) GS2_TRY_HIP(hipMemcpyAsync(&stats[q], dev, sizeof(PartStats), hipMemcpyDeviceToHost, s));
    }
    GS2_TRY_HIP(hipStreamSynchronize(s));
    size_t bytes = 0, at[3][3];
    for (int q = 0; q < np; ++q) {
        Sell &S = *part[first + q];
        S.padded = ends[q];
        S.nnz = (int64_t)stats[q].total;
        // padding sits at offset 0, and past the last row as far below it as the
        // last slice goes on
        const int64_t lo = std::min<int64_t>(stats[q].lo, n - ns * C), hi = stats[q].hi;
        const bool narrow = S.nnz > 0 && hi - lo <= 65535;
        S.off_min = narrow ? (int)lo : 0;
        const size_t cnt = (size_t)std::max<int64_t>(S.padded, WAVE);
        at[q][0] = bytes;
        at[q][1] = at[q][0] + aligned(cnt * sizeof(int32_t));
        at[q][2] = at[q][1] + aligned(cnt * vb);
        bytes = at[q][2] + (narrow ? aligned(cnt * sizeof(uint16_t)) : 0);
        S.off = narrow ? (uint16_t *)1 : nullptr; // placed below
    }
    GS2_TRY_HIP(hipMalloc(&own.mem[1], bytes));
    for (int q = 0; q < np; ++q) {
        Sell &S = *part[first + q];
        char *m = (char *)own.mem[1];
        S.col = (int32_t *)(m + at[q][0]);
        S.val = m + at[q][1];
        if (S.off) S.off = (uint16_t *)(m + at[q][2]);
        if (h.precision == GS2_FP64) fill_part<double>(h, S, first + q, R, A, sc.err, s);
        else if (h.precision == GS2_FP32) fill_part<float>(h, S, first + q, R, A, sc.err, s);
        else fill_part<_Float16>(h, S, first + q, R, A, sc.err, s);
    }
    GS2_TRY_HIP(hipGetLastError());
    return GS2_OK;
}

static int build_triangles(Handle &h, int K, const gs2_csr &A, const SetupScratch &sc, hipStream_t s)
{
    GS2_TRY(build_parts(h, PART_L, PART_U, K, A, sc, s));
    h.L.nt = h.U.nt = h.L.stored_bytes() + h.U.stored_bytes() > NT_TRIANGLES_BYTES ? 1 : 0;
    return GS2_OK;
}

// The setup's flush buffer (FLUSH_BYTES of zeros, read before each timed
// pass), held for the timing and released when the setup returns.  Without
// memory for it the passes are timed back to back.
struct FlushBuffer {
    Handle &h;
    hipStream_t s;
    FlushBuffer(Handle &hh, hipStream_t ss) : h(hh), s(ss) {}
    // called where a timing begins
    void hold()
    {
        if (h.flush) return;
        if (hipMalloc(&h.flush, FLUSH_BYTES) != hipSuccess) {
            h.flush = nullptr;
            (void)hipGetLastError();
            return;
        }
        if (hipMemsetAsync(h.flush, 0, FLUSH_BYTES, s) != hipSuccess) {
            (void)hipFree(h.flush);
            h.flush = nullptr;
            (void)hipGetLastError();
        }
    }
    ~FlushBuffer()
    {
        if (h.flush) (void)hipFree(h.flush);
        h.flush = nullptr;
    }
};

// Schedules of the diagonal layout chosen by timing (packed into one number).
struct DiaChoice {
    int fmt, R, lds, remap, b3;
    int pack() const { return fmt | R << 4 | lds << 8 | remap << 9 | b3 << 10; }
    static DiaChoice unpack(int v) { return DiaChoice{v & 15, v >> 4 & 15, v >> 8 & 1, v >> 9 & 1, v >> 10 & 1}; }
};

// Decide the layout of the GS2 / JR passes: keep the sliced-ELL triangles, or
// build diagonal-interleaved copies (Dia: scalar diagonals, or 3-row blocks
// along node offsets) and time them against sliced ELL.
static int choose_format(Handle &h, const gs2_csr &A, const gs2_options &o, SetupScratch &sc, FlushBuffer &flush,
                         hipStream_t s, bool can_time, const std::string &key_base)
{
    h.fmt = FMT_SELL;
    h.lds = 0;
    h.tuned = 0;
    if (o.format == GS2_FORMAT_SELL) return GS2_OK;
    // the automatic choice is made by timing only; without it sliced ELL stays
    if (o.format == GS2_FORMAT_AUTO && !(can_time && o.autotune)) return GS2_OK;
    const int64_t n = h.n;
    const bool any = h.blocks == 1 && n > 0 && n <= (int64_t(1) << 30);
    std::vector<int> offL, offU;
    const std::vector<int> &boffL = sc.pat.bl, &boffU = sc.pat.bu;
    const int64_t nnzL = sc.pat.nl, nnzU = sc.pat.nu;
    bool dia_ok = false, b3_ok = false;
    if (any) {
        // stored diagonal entries (padding included) at most 1.5x the real ones
        auto fits = [n](const std::vector<int> &off, int64_t nnz, double rows) {
            return (int)off.size() <= DIA_MAX && rows * off.size() * n <= 1.5 * nnz + rows * 64.0 * off.size();
        };
        if (o.format != GS2_FORMAT_BLOCK3 && !sc.pat.many_d) {
            for (int d : sc.pat.d)
                if (d) (d < 0 ? offL : offU).push_back(d);
            dia_ok = fits(offL, nnzL, 1.0) && fits(offU, nnzU, 1.0);
        }
        if (!dia_ok && o.format != GS2_FORMAT_DIA && !sc.pat.many_b)
            b3_ok = fits(boffL, nnzL, 3.0) && fits(boffU, nnzU, 3.0);
    }
    h.DL.ndiag = dia_ok ? (int)offL.size() : b3_ok ? (int)boffL.size() : 0;
    h.DU.ndiag = dia_ok ? (int)offU.size() : b3_ok ? (int)boffU.size() : 0;
    if (!dia_ok && !b3_ok) return o.format == GS2_FORMAT_AUTO ? GS2_OK : GS2_ERR_ARG;
    const int b3 = dia_ok ? 0 : 1; // the one diagonal kind this pattern admits
    const int vb = h.precision == GS2_FP64 ? 8 : h.precision == GS2_FP32 ? 4 : 2;
    std::vector<int> Rs, ldss;
    for (int R = 1; R <= 8; R *= 2)
        if (R * vb >= 2 && R * vb <= 16 && (o.rows_per_lane == 0 || o.rows_per_lane == R)) Rs.push_back(R);
    if (Rs.empty()) return GS2_ERR_ARG; // a forced rows-per-lane whose load is not 2..16 bytes
    // the block passes try the widest load first: a narrower one must then win
    // by the margin below (the float64 elasticity passes at two nodes per lane
    // ran 10 % faster in the solve than at one, while the timed pair of passes
    // often put the two within the margin)
    if (b3) std::reverse(Rs.begin(), Rs.end());
    if (b3) ldss = {0}; // block passes read their source directly
    else if (o.lds_staging == 0) ldss = {0, 1};
    else ldss = {o.lds_staging == 2 ? 1 : 0};
    std::vector<int> rms;
    if (o.xcd_ranges == 0) rms = {1, 0};
    else rms = {o.xcd_ranges == 2 ? 1 : 0};
    // both triangles, in one allocation
    auto build = [&](int R) -> int {
        free_dia(h.DL);
        free_dia(h.DU);
        const size_t bl = shape_dia(h.DL, n, h.precision, R, b3 ? boffL : offL, nnzL, b3);
        const size_t bu = shape_dia(h.DU, n, h.precision, R, b3 ? boffU : offU, nnzU, b3);
        GS2_TRY_HIP(hipMalloc(&h.DL.mem, bl + bu));
        GS2_TRY_HIP(hipMemsetAsync(h.DL.mem, 0, bl + bu, s));
        h.DL.val = h.DL.mem;
        h.DU.val = (char *)h.DL.mem + bl;
        for (int lower = 1; lower >= 0; --lower) {
            const Dia &D = lower ? h.DL : h.DU;
            if (h.precision == GS2_FP64) fill_dia<double>(D, n, lower, A, sc.lcnt, h.sl, h.sr, sc.err, s);
            else if (h.precision == GS2_FP32) fill_dia<float>(D, n, lower, A, sc.lcnt, h.sl, h.sr, sc.err, s);
            else fill_dia<_Float16>(D, n, lower, A, sc.lcnt, h.sl, h.sr, sc.err, s);
        }
        GS2_TRY_HIP(hipGetLastError());
        h.DL.nt = h.DU.nt = h.DL.stored_bytes() + h.DU.stored_bytes() > NT_TRIANGLES_BYTES ? 1 : 0;
        return GS2_OK;
    };
    const bool timed = can_time && o.autotune &&
                       (o.format == GS2_FORMAT_AUTO || Rs.size() > 1 || ldss.size() > 1 || rms.size() > 1);
    if (!timed) {
        if (o.format == GS2_FORMAT_AUTO) return GS2_OK; // untimed automatic choice: sliced ELL
        GS2_TRY(build(*std::max_element(Rs.begin(), Rs.end()))); // forced: the widest load allowed
        h.fmt = FMT_DIA;
        h.lds = ldss.back();
        h.remap = rms.front();
        return GS2_OK;
    }
    char kb[56];
    std::snprintf(kb, sizeof kb, "_d%d_%d_b%d_f%d_r%d_s%d_x%d", h.DL.ndiag, h.DU.ndiag, b3, o.format, o.rows_per_lane,
                  o.lds_staging, o.xcd_ranges);
    const std::string key = key_base + kb;
    DiaChoice ch{FMT_SELL, 0, 0, 1, 0};
    int packed = 0;
    if (choice_get(key, &packed)) {
        ch = DiaChoice::unpack(packed);
    } else {
        flush.hold();
        float best = 1e30f;
        if (o.format == GS2_FORMAT_AUTO) {
            h.fmt = FMT_SELL;
            GS2_TRY(time_inner_pass(h, s, &best, true));
        }
        for (int R : Rs) {
            GS2_TRY(build(R));
            for (int l : ldss)
                for (int rm : rms) { // workgroups walked per XCD, or in dispatch order
                    h.fmt = FMT_DIA;
                    h.lds = l;
                    h.remap = rm;
                    float ms = 0.f;
                    GS2_TRY(time_inner_pass(h, s, &ms, true));
                    // a new candidate must win by more than the timing noise
                    if (ms < 0.97f * best) {
                        best = ms;
                        ch = DiaChoice{FMT_DIA, R, l, rm, b3};
                    }
                }
        }
        choice_put(key, ch.pack());
    }
    h.tuned = 1;
    if (ch.fmt == FMT_SELL) {
        h.fmt = FMT_SELL;
        h.lds = 0;
        free_dia(h.DL);
        free_dia(h.DU);
        return GS2_OK;
    }
    if (!h.DL.val || h.DL.R != ch.R) GS2_TRY(build(ch.R));
    h.fmt = FMT_DIA;
    h.lds = ch.lds;
    h.remap = ch.remap;
    return GS2_OK;
}

static int read_err(int *err, hipStream_t s)
{
    int f = 0;
    GS2_TRY_HIP(hipMemcpyAsync(&f, err, sizeof(int), hipMemcpyDeviceToHost, s));
    GS2_TRY_HIP(hipStreamSynchronize(s));
    return flags_to_status(f);
}

void free_perm(Perm &P)
{
    for (void *p : {(void *)P.rows, P.val}) // the others lie behind these
        if (p) (void)hipFree(p);
    P = Perm{};
}

// Stored entries of each chunk: 64 times the longest of its rows (off-diagonal
// entries); zero at index nchunks, so that an exclusive scan yields the end.  And
// the most main entries of its rows.
__global__ __launch_bounds__(256) void k_perm_len(int64_t nchunks, const int32_t *__restrict__ rows,
                                                  const int32_t *__restrict__ rp, const int32_t *__restrict__ lcnt,
                                                  int lower, int64_t *__restrict__ len, int32_t *__restrict__ mains)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t c = g / WAVE;
    if (c > nchunks) return;
    const int i = c < nchunks ? rows[g] : -1;
    int m = i < 0 ? 0 : rp[i + 1] - rp[i] - 1;
    int mc = i < 0 ? 0 : lower ? lcnt[i] : m - lcnt[i];
    for (int o = 1; o < WAVE; o <<= 1) {
        m = max(m, __shfl_xor(m, o));
        mc = max(mc, __shfl_xor(mc, o));
    }
    if (g % WAVE == 0) {
        len[c] = (int64_t)WAVE * m;
        if (mains && c < nchunks) mains[c] = mc;
    }
}

// One workgroup per chunk, a thread per position and every fourth entry: the row's
// entries, the main triangle's first (lower = 1: the lower triangle is the main
// one), scaled and rounded as in k_fill.  A main entry's column goes through `place` when it is given.
template <typename VT>
__global__ __launch_bounds__(256) void k_perm_fill(const int32_t *__restrict__ rows,
                                                   const int64_t *__restrict__ ptr, const int32_t *__restrict__ rp,
                                                   const int32_t *__restrict__ ci, const double *__restrict__ va,
                                                   const int32_t *__restrict__ lcnt, int lower,
                                                   const int32_t *__restrict__ place,
                                                   const double *__restrict__ sl, const double *__restrict__ sr,
                                                   int32_t *__restrict__ col, uint16_t *__restrict__ off, int off_min,
                                                   VT *__restrict__ val)
{
    const int64_t c = blockIdx.x;
    const int ln = threadIdx.x % WAVE;
    const int i = rows[c * WAVE + ln];
    const int64_t beg = ptr[c];
    const int steps = (int)((ptr[c + 1] - beg) / WAVE);
    const int b = i < 0 ? 0 : rp[i], lc = i < 0 ? 0 : lcnt[i], tot = i < 0 ? 0 : rp[i + 1] - b - 1, uc = tot - lc;
    const int mc = lower ? lc : uc;
    const double srow = i < 0 ? 0.0 : sl[i];
    int ovf = 0; // the natural-order triangles report it
    for (int t = threadIdx.x / WAVE; t < steps; t += 256 / WAVE) {
        const int64_t pos = beg + (int64_t)t * WAVE + ln;
        if (t >= tot) {
            if (off) off[pos] = PERM_PAD16;
            else col[pos] = PERM_PAD;
            val[pos] = VT(0);
            continue;
        }
        const bool low = lower ? t < mc : t >= mc;
        const int k = b + (low ? (lower ? t : t - mc) : lc + 1 + (lower ? t - mc : t));
        const int j = ci[k];
        if (off) off[pos] = (uint16_t)(j - i - off_min);
        else col[pos] = t >= mc ? ~j : place ? place[j] : j;
        val[pos] = convert_scaled<VT>((srow * va[k]) * sr[j], &ovf);
    }
}

// The rows in the given order (-1: no row), 64 per chunk, with their entries;
// by_place: the main entries name positions of this order instead of rows; mains,
// if not null: the chunks' longest main parts;
// span: the pattern's smallest and largest col - row, for 16-bit offsets where
// they fit (null: columns).
static int build_perm(Handle &h, Perm &P, std::vector<int32_t> &order, int lower, bool by_place, const gs2_csr &A,
                      const int32_t *lcnt, const Pattern *span, int32_t **mains, hipStream_t s)
{
    // three allocations (0.1 ms each): what stays of the rows, what stays of their
    // entries, and what goes with this scope
    struct Tmp {
        int64_t *len = nullptr;
        int32_t *place = nullptr;
        ~Tmp()
        {
            if (len) (void)hipFree(len);
        }
    } tmp;
    std::vector<int32_t> place(by_place ? h.n : 0);
    if (by_place)
        for (size_t q = 0; q < order.size(); ++q)
            if (order[q] >= 0) place[order[q]] = (int32_t)q;
    order.resize((order.size() + WAVE - 1) / WAVE * WAVE, -1);
    P.nchunks = (int64_t)order.size() / WAVE;
    int64_t total = 0;
    const size_t lens = aligned(sizeof(int64_t) * (P.nchunks + 1 + scan_tmp(P.nchunks + 1)));
    GS2_TRY_HIP(hipMalloc(&tmp.len, lens + sizeof(int32_t) * place.size()));
    if (by_place) {
        tmp.place = (int32_t *)((char *)tmp.len + lens);
        GS2_TRY_HIP(hipMemcpyAsync(tmp.place, place.data(), sizeof(int32_t) * place.size(), hipMemcpyHostToDevice, s));
    }
    const size_t rb = aligned(sizeof(int32_t) * order.size()), pb = aligned(sizeof(int64_t) * (P.nchunks + 1));
    GS2_TRY_HIP(hipMalloc(&P.rows, rb + pb + (mains ? sizeof(int32_t) * P.nchunks : 0)));
    P.ptr = (int64_t *)((char *)P.rows + rb);
    if (mains) *mains = (int32_t *)((char *)P.rows + rb + pb);
    GS2_TRY_HIP(hipMemcpyAsync(P.rows, order.data(), sizeof(int32_t) * order.size(), hipMemcpyHostToDevice, s));
    k_perm_len<<<(unsigned)(((P.nchunks + 1) * WAVE + 255) / 256), 256, 0, s>>>(P.nchunks, P.rows, A.rowptr, lcnt, lower,
                                                                                   tmp.len, mains ? *mains : nullptr);
    GS2_TRY(exclusive_scan_i64(tmp.len, P.ptr, P.nchunks + 1, tmp.len + P.nchunks + 1, s));
    GS2_TRY_HIP(hipMemcpyAsync(&total, P.ptr + P.nchunks, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    GS2_TRY_HIP(hipStreamSynchronize(s)); // `order` and `place` may go
    const size_t vb = h.precision == GS2_FP64 ? 8 : h.precision == GS2_FP32 ? 4 : 2;
    const size_t cnt = (size_t)std::max<int64_t>(total, WAVE), vals = aligned(vb * cnt);
    const bool narrow = span && (int64_t)span->hi - span->lo < PERM_PAD16;
    GS2_TRY_HIP(hipMalloc(&P.val, vals + (narrow ? sizeof(uint16_t) : sizeof(int32_t)) * cnt));
    if (narrow) {
        P.off_min = span->lo;
        P.off = (uint16_t *)((char *)P.val + vals);
    } else {
        P.col = (int32_t *)((char *)P.val + vals);
    }
    const unsigned g = (unsigned)P.nchunks;
    if (h.precision == GS2_FP64)
        k_perm_fill<double><<<g, 256, 0, s>>>(P.rows, P.ptr, A.rowptr, A.colind, A.val, lcnt, lower,
                                              tmp.place, h.sl, h.sr, P.col, P.off, P.off_min, (double *)P.val);
    else if (h.precision == GS2_FP32)
        k_perm_fill<float><<<g, 256, 0, s>>>(P.rows, P.ptr, A.rowptr, A.colind, A.val, lcnt, lower,
                                             tmp.place, h.sl, h.sr, P.col, P.off, P.off_min, (float *)P.val);
    else
        k_perm_fill<_Float16><<<g, 256, 0, s>>>(P.rows, P.ptr, A.rowptr, A.colind, A.val, lcnt, lower,
                                                tmp.place, h.sl, h.sr, P.col, P.off, P.off_min, (_Float16 *)P.val);
    GS2_TRY_HIP(hipGetLastError());
    GS2_TRY_HIP(hipStreamSynchronize(s)); // tmp goes with this scope
    return GS2_OK;
}

// Multicolor ordering (Section 6, multi-threaded Gauss-Seidel): greedy first
// fit in natural row order on the symmetrised pattern; a row takes the
// smallest color not held by an earlier row it is coupled to (a_ij or a_ji
// nonzero).  Rows are then grouped color by color, each color from a chunk
// of its own.
static int build_colors(Handle &h, const gs2_csr &A, const int32_t *lcnt, const std::vector<int32_t> &rp,
                        const std::vector<int32_t> &ci, const Pattern &span, hipStream_t s)
{
    const int64_t n = h.n;
    // transpose pattern (column -> rows), to see couplings a_ji from earlier rows j
    std::vector<int32_t> tp(n + 1, 0), tc(std::max<size_t>(ci.size(), 1));
    for (int64_t i = 0; i < n; ++i)
        for (int32_t k = rp[i]; k < rp[i + 1]; ++k) tp[ci[k] + 1]++;
    for (int64_t i = 0; i < n; ++i) tp[i + 1] += tp[i];
    std::vector<int32_t> fill(tp.begin(), tp.end() - 1);
    for (int64_t i = 0; i < n; ++i)
        for (int32_t k = rp[i]; k < rp[i + 1]; ++k) tc[fill[ci[k]]++] = (int32_t)i;
    std::vector<int32_t> color(n), seen(n + 2, -1);
    std::vector<int64_t> cnt, nnz;
    int ncol = 0;
    for (int64_t i = 0; i < n; ++i) {
        for (int32_t k = rp[i]; k < rp[i + 1]; ++k)
            if (ci[k] < i) seen[color[ci[k]]] = (int32_t)i;
        for (int32_t k = tp[i]; k < tp[i + 1]; ++k)
            if (tc[k] < i) seen[color[tc[k]]] = (int32_t)i;
        int c = 0;
        while (seen[c] == i) ++c;
        color[i] = c;
        if (c == ncol) {
            ++ncol;
            cnt.push_back(0);
            nnz.push_back(0);
        }
        cnt[c]++;
        nnz[c] += rp[i + 1] - rp[i] - 1;
    }
    std::vector<int64_t> ptr(ncol + 1, 0), pos(ncol);
    for (int c = 0; c < ncol; ++c) {
        pos[c] = ptr[c] * WAVE;
        ptr[c + 1] = ptr[c] + (cnt[c] + WAVE - 1) / WAVE;
    }
    std::vector<int32_t> rows(ptr[ncol] * WAVE, -1);
    for (int64_t i = 0; i < n; ++i) rows[pos[color[i]]++] = (int32_t)i;
    GS2_TRY(build_perm(h, h.PC, rows, 1, false, A, lcnt, &span, nullptr, s));
    h.ncolors = ncol;
    h.color_ptr = std::move(ptr);
    h.color_rows = std::move(cnt);
    h.color_nnz = std::move(nnz);
    return GS2_OK;
}

// Level sets of the DAGs of L (ascending) and U (descending), computed on the
// host from a copy of the pattern: level_i = 1 + max level over the
// triangle's entries of row i.  Rows are then grouped level by level.
static int build_levels(Handle &h, const gs2_csr &A, const int32_t *lcnt, const Pattern &span, hipStream_t s)
{
    const int64_t n = A.n;
    std::vector<int32_t> rp(n + 1), ci(A.nnz);
    GS2_TRY_HIP(hipMemcpyAsync(rp.data(), A.rowptr, sizeof(int32_t) * (n + 1), hipMemcpyDeviceToHost, s));
    if (A.nnz) GS2_TRY_HIP(hipMemcpyAsync(ci.data(), A.colind, sizeof(int32_t) * A.nnz, hipMemcpyDeviceToHost, s));
    GS2_TRY_HIP(hipStreamSynchronize(s));
    GS2_TRY_HIP(hipMalloc(&h.tri_next, 3 * sizeof(unsigned)));
    std::vector<int32_t> lev(n);
    for (int lower = 1; lower >= 0; --lower) {
        int nlev = 0;
        for (int64_t q = 0; q < n; ++q) {
            const int64_t i = lower ? q : n - 1 - q;
            int lv = 0;
            for (int32_t k = rp[i]; k < rp[i + 1]; ++k) {
                const int32_t c = ci[k];
                if (lower ? c < i : c > i) lv = std::max(lv, lev[c] + 1);
            }
            lev[i] = lv;
            nlev = std::max(nlev, lv + 1);
        }
        std::vector<int64_t> pos(nlev + 1, 0);
        for (int64_t i = 0; i < n; ++i) pos[lev[i] + 1]++;
        for (int l = 0; l < nlev; ++l) pos[l + 1] += pos[l];
        std::vector<int32_t> rows(n);
        for (int64_t i = 0; i < n; ++i) rows[pos[lev[i]]++] = (int32_t)i;
        GS2_TRY(build_perm(h, lower ? h.PL : h.PU, rows, lower, true, A, lcnt, nullptr,
                           span.maxlen <= 8 ? nullptr : lower ? &h.mains_l : &h.mains_u, s));
        (lower ? h.nlev_l : h.nlev_u) = nlev;
    }
    return build_colors(h, A, lcnt, rp, ci, span, s);
}

// The scaling vectors and, with work, the applies' temporaries.
static int alloc_vectors(Handle &h, bool work, hipStream_t s)
{
    const size_t n = (size_t)std::max<int64_t>(h.n, 1), d = aligned(sizeof(double) * n);
    const size_t vb = aligned(prec_bytes(h.precision) * n);
    const bool sv = h.precision != GS2_FP64, yh = h.blocks > 1;
    const size_t small = work ? small_bytes(h) : 0;
    GS2_TRY_HIP(hipMalloc(&h.vec, 2 * d + (work ? (5 + sv + yh) * vb : 0) + small));
    char *p = (char *)h.vec;
    h.sl = (double *)p;
    h.sr = (double *)(p + d);
    if (!work) return GS2_OK;
    p += 2 * d;
    for (void **q : {&h.xh, &h.xh2, &h.rh, &h.ga, &h.gb}) {
        *q = p;
        p += vb;
    }
    if (sv) {
        h.sv = p;
        p += vb;
    }
    if (yh) {
        h.yh = p;
        p += vb;
    }
    if (small) small_init(h, p, s);
    return GS2_OK;
}

int setup_handle(Handle &h, const gs2_csr &A, const gs2_options &o, hipStream_t s, bool alloc_vecs)
{
    const int64_t n = A.n;
    if (n == 0) return GS2_OK;
    SetupScratch sc;
    GS2_TRY(sc.alloc(n));
    GS2_TRY(alloc_vectors(h, alloc_vecs, s));
    GS2_TRY_HIP(hipMemsetAsync(sc.err, 0, sizeof(int), s));
    GS2_TRY(scan_pattern(A, sc.lcnt, sc.ucnt, h.sl, h.sr, sc.dev, sc.pat, s));
    GS2_TRY(flags_to_status(sc.pat.err));

    if (!small_suits(h, sc.pat)) h.ep = nullptr; // pass by pass
    // row-length statistics of L (U has the same count for symmetric patterns)
    const double avg = n ? (double)(A.nnz - n) / (2.0 * n) : 0.0;
    const int maxlen = sc.pat.maxlen;
    const std::string shape = shape_key(n, avg, maxlen, h.precision);

    int K = o.lanes_per_row;
    if (K != 0 && (K < 1 || K > 64 || (K & (K - 1)))) return GS2_ERR_ARG;
    const bool can_time = alloc_vecs && n >= 4096;
    // the schedule timing below reads the flush buffer before each timed pass
    FlushBuffer flush(h, s);
    if (K == 0) {
        K = choose_lanes(avg, maxlen);
        if (o.autotune && can_time && !choice_get("K_" + shape, &K)) {
            flush.hold();
            float best = 1e30f;
            // each candidate is timed on one inner pass over L and one residual pass
            // over L and U, with the cache policy its stored size implies
            for (int cand = 1; cand <= 16; cand *= 2) {
                if (cand > 1 && cand > 2 * std::max(1.0, avg)) break;
                GS2_TRY(build_triangles(h, cand, A, sc, s));
                float ms = 0.f;
                GS2_TRY(time_inner_pass(h, s, &ms, true));
                // a wider candidate must win by more than the timing noise
                if (ms < 0.97f * best) { best = ms; K = cand; }
            }
            choice_put("K_" + shape, K);
        }
    }
    GS2_TRY(build_triangles(h, K, A, sc, s));
    GS2_TRY(choose_format(h, A, o, sc, flush, s, can_time, shape));
    if (h.blocks > 1) GS2_TRY(build_parts(h, PART_E, PART_E, K, A, sc, s));
    GS2_TRY(read_err(sc.err, s));
    if (o.build_levels) GS2_TRY(build_levels(h, A, sc.lcnt, sc.pat, s));
    GS2_TRY_HIP(hipStreamSynchronize(s));
    return GS2_OK;
}

} // namespace gs2

using namespace gs2;

Handle::~Handle()
{
    free_sell(L);
    free_sell(U);
    free_sell(E);
    free_dia(DL);
    free_dia(DU);
    free_perm(PL);
    free_perm(PU);
    free_perm(PC);
    for (void *p : {vec, (void *)tri_next})
        if (p) (void)hipFree(p);
    if (gw) free_gmres_work(gw);
    if (cw) free_cg_work(cw);
}

extern "C" {

void gs2_default_options(gs2_options *opt)
{
    if (!opt) return;
    opt->precision = GS2_FP64;
    opt->inner_damping = 1.0;
    opt->compact = 0;
    opt->build_levels = 0;
    opt->autotune = 1;
    opt->lanes_per_row = 0;
    opt->rhs_per_item = 0;
    opt->orthogonalization = 0;
    opt->blocks = 1;
    opt->local_sweeps = 1;
    opt->team_rows = 0;
    opt->team_wait_ms = 0;
    opt->format = GS2_FORMAT_AUTO;
    opt->rows_per_lane = 0;
    opt->lds_staging = 0;
    opt->stagnation_cycles = 0;
    opt->spmv_format = GS2_FORMAT_AUTO;
    opt->basis_loads = 0;
    opt->xcd_ranges = 0;
}

int gs2_setup(const gs2_csr *A, int sweeps, int inner, double damping, int variant, const gs2_options *opt,
              void *stream, gs2_handle **out)
{
    if (!out) return GS2_ERR_ARG;
    *out = nullptr;
    if (!A || A->n < 0 || A->n >= (int64_t(1) << 31) - 1 || A->nnz < A->n || A->nnz >= (int64_t(1) << 31) - 1)
        return GS2_ERR_ARG;
    if ((A->n > 0) && (!A->rowptr || !A->colind || !A->val)) return GS2_ERR_ARG;
    if (sweeps < 1 || inner < 0 || variant < GS2_FORWARD || variant > GS2_SYMMETRIC) return GS2_ERR_ARG;
    if (!(damping > 0.0 && damping < 2.0)) return GS2_ERR_ARG;
    gs2_options o;
    gs2_default_options(&o);
    if (opt) o = *opt;
    if (o.precision < GS2_FP64 || o.precision > GS2_FP16_SCALED) return GS2_ERR_ARG;
    if (o.orthogonalization < 0 || o.orthogonalization > 1) return GS2_ERR_ARG;
    if (o.blocks < 0 || o.local_sweeps < 0 || (o.blocks > 1 && (o.compact || o.build_levels)) ||
        (int64_t)o.blocks > std::max<int64_t>(A->n, 1))
        return GS2_ERR_ARG;
    if (!(o.inner_damping > 0.0 && o.inner_damping <= 2.0)) return GS2_ERR_ARG;
    if (o.format < GS2_FORMAT_AUTO || o.format > GS2_FORMAT_BLOCK3 || o.rows_per_lane < 0 || o.lds_staging < 0 ||
        o.lds_staging > 2 || o.spmv_format < GS2_FORMAT_AUTO || o.spmv_format > GS2_FORMAT_BLOCK3 || o.xcd_ranges < 0 ||
        o.xcd_ranges > 2 || o.basis_loads < 0 || o.basis_loads > 2)
        return GS2_ERR_ARG;
    gs2_handle *H = new (std::nothrow) gs2_handle;
    if (!H) return GS2_ERR_NOMEM;
    Handle &h = H->h;
    h.n = A->n;
    h.sweeps = sweeps;
    h.inner = inner;
    h.variant = variant;
    h.omega = damping;
    h.gamma = o.inner_damping;
    h.compact = o.compact ? 1 : 0;
    h.orth = o.orthogonalization;
    h.stag_cycles = o.stagnation_cycles;
    h.spmv_fmt = o.spmv_format;
    h.basis_req = o.basis_loads;
    h.blocks = std::max(1, o.blocks);
    h.local_sweeps = std::max(1, o.local_sweeps);
    h.precision = o.precision;
    hipStream_t s = (hipStream_t)stream;
    // resolve the allocation-free entry point's scratch on this device now
    // (cached per device; should it fail, that entry point reports it)
    (void)noalloc_scratch(nullptr);
    int st = GS2_ERR_HIP;
    try {
        st = setup_handle(h, *A, o, s, true);
    } catch (const std::bad_alloc &) {
        st = GS2_ERR_NOMEM;
    } catch (...) {
        st = GS2_ERR_HIP;
    }
    if (st != GS2_OK) {
        (void)hipStreamSynchronize(s);
        delete H;
        return st;
    }
    *out = H;
    return GS2_OK;
}

void gs2_destroy(gs2_handle *H)
{
    if (!H) return;
    (void)hipDeviceSynchronize();
    delete H;
}

const char *gs2_status_string(int status)
{
    switch (status) {
    case GS2_OK: return "success";
    case GS2_ERR_ARG: return "invalid argument";
    case GS2_ERR_BAD_CSR: return "malformed CSR (unsorted, duplicate or out-of-range column, bad row pointer)";
    case GS2_ERR_ZERO_DIAG: return "diagonal entry missing or zero";
    case GS2_ERR_NONFINITE: return "non-finite value (NaN or Inf)";
    case GS2_ERR_NOMEM: return "device allocation failed";
    case GS2_ERR_HIP: return "HIP runtime error";
    case GS2_ERR_FP16_RANGE: return "scaled matrix value outside binary16 range";
    case GS2_ERR_NO_LEVELS: return "handle was built without level sets";
    case GS2_ERR_SCRATCH: return "input exceeds the fixed scratch of the allocation-free entry point";
    case GS2_NOT_CONVERGED: return "not converged within maxit iterations";
    case GS2_BREAKDOWN_EXACT: return "GMRES exact breakdown (singular Hessenberg)";
    case GS2_STAGNATED: return "GMRES stagnated (true residual not halved over the stagnation window)";
    default: return "unknown status";
    }
}

int gs2_handle_query(const gs2_handle *H, int64_t *n, int64_t *nnz_l, int64_t *nnz_u, int64_t *bytes_stored,
                     int *lanes_per_row, int *levels_l, int *levels_u)
{
    if (!H) return GS2_ERR_ARG;
    const Handle &h = H->h;
    if (n) *n = h.n;
    if (nnz_l) *nnz_l = h.L.nnz;
    if (nnz_u) *nnz_u = h.U.nnz;
    if (bytes_stored)
        *bytes_stored = (h.L.padded + h.U.padded) * (int64_t)(4 + h.L.val_bytes) +
                        h.L.padded * (h.L.off ? 2 : 0) + h.U.padded * (h.U.off ? 2 : 0) +
                        8 * (h.L.nslices + h.U.nslices + 2) + 16 * h.n;
    if (lanes_per_row) *lanes_per_row = h.L.K;
    if (levels_l) *levels_l = h.nlev_l;
    if (levels_u) *levels_u = h.nlev_u;
    return GS2_OK;
}

int gs2_handle_schedule(const gs2_handle *H, int *format, int *lanes_per_row, int *rows_per_lane, int *vector_bytes,
                        int *lds_staging, int *xcd_ranges, int *ndiag_l, int *ndiag_u, int *tuned)
{
    if (!H) return GS2_ERR_ARG;
    const Handle &h = H->h;
    const bool dia = h.fmt == FMT_DIA;
    if (format) *format = !dia ? GS2_FORMAT_SELL : h.DL.b3 ? GS2_FORMAT_BLOCK3 : GS2_FORMAT_DIA;
    if (lanes_per_row) *lanes_per_row = h.L.K;
    if (rows_per_lane) *rows_per_lane = dia ? h.DL.R : 0;
    if (vector_bytes) *vector_bytes = dia ? h.DL.R * h.DL.val_bytes : 0;
    if (lds_staging) *lds_staging = dia ? h.lds : 0;
    if (xcd_ranges) *xcd_ranges = dia ? h.remap : 0;
    if (ndiag_l) *ndiag_l = h.DL.ndiag;
    if (ndiag_u) *ndiag_u = h.DU.ndiag;
    if (tuned) *tuned = h.tuned;
    return GS2_OK;
}

} // extern "C"
