// A GS2 / JR apply of a small system in one launch.
//
// Launched pass by pass an apply of a few thousand rows is the host's time to
// enqueue its launches, or 4 to 5 us for each of them.  Here a wavefront keeps
// its 64 rows through all passes, a thread per row, with the row's first
// entries of both triangles in registers, and waits for nothing but the values
// its rows' columns name.
//
// Every vector that a pass gathers and another pass writes has a buffer of
// its own, in which an unknown is its own flag, as in the exact sweeps: it
// starts as a NaN pattern no result keeps, is stored and read at agent scope
// (past the caches that XCDs do not share), and a thread polls until the
// entries it needs are there: one trip for flag and value, 0.55 us from store
// to load.  There are two sets of buffers; an apply uses one and resets the
// other, on which nothing runs any more, for the next apply.  Which set is in
// turn is counted per wavefront on the device, so that an apply replayed from
// a graph takes its turn too.
//
// The wavefronts wait for each other, so all of an apply have to run at once:
// SMALL_MAX_N rows are SMALL_MAX_N / 64 wavefronts of at most 128 registers, of
// which the chip holds 4096; other kernels only delay that.  The waits are
// bounded all the same (the pattern then passes on as NaN).
//
// Sums, roundings and therefore every bit are those of the passes launched one
// by one (sweep.hip: Launch::gs2 and Launch::jr), for which fused operations
// are written out where the compiler could fuse another pair.
//
// Enqueued one after the other, SGS2(1,1) in float64 (a call, in us): 11.6
// pass by pass and 6.5 in one launch on 64 x 64 points, 11.9 and 6.8 on 256 x
// 256; GS2(2,2) in float32 19.6 and 7.4, 19.2 and 8.5.  What is left is the
// host's time to enqueue one launch.  More rows would gain too, but wavefronts
// that wait for each other have to fit next to those of other streams.
#include <algorithm>

#include "gs2_internal.hpp"
#include "resident.hpp"

namespace gs2 {

namespace {

// Looks before a wait is given up, half a microsecond or more each (counted, not
// timed: a process that shares the device may be set aside for any time).
constexpr unsigned SMALL_WAIT_POLLS = 1u << 22;
constexpr int SMALL_LANES = 4; // most lanes per row whose sums are repeated

struct SmallArgs {
    const int *stop;
    int n, ne;
    int jr, sweeps, inner, variant, compact;
    double omega, gamma;
    ResSell L, U;
    const double *sl, *sr, *v;
    double *z;
    void *ex;     // two sets of ne vectors
    unsigned *ep; // applies done, per wavefront
};

template <typename VT, typename AT, int KL>
struct SmallRow {
    using BT = typename Bits<AT>::T;
    static constexpr BT NR = Bits<AT>::not_ready;
    static constexpr int U = 4; // entries of a row taken at a time
    static_assert(U % (1 << KL) == 0, "an entry's lane follows from its place among the U");

    const SmallArgs &a;
    int row;
    bool own;

    // a triangle's row: entry k at p = at + (k >> lk) 64 + (k mod 2^lk), the
    // first U of them held (the last one repeated where there are fewer)
    struct Row {
        const int32_t *col;
        const VT *val;
        int lk, at, cnt;
        int c[U];
        VT v[U];
    };
    __device__ void fetch(const Row &R, int e, int *c, VT *v) const
    {
        const int km = (1 << R.lk) - 1;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int k = e + q < R.cnt ? e + q : R.cnt - 1;
            const int p = R.at + (k >> R.lk) * WAVE + (k & km);
            c[q] = R.col[p];
            v[q] = R.val[p];
        }
    }
    __device__ void load(Row &R, const ResSell &T) const
    {
        R.col = T.col;
        R.val = (const VT *)T.val;
        R.lk = T.lk;
        R.cnt = 0;
        R.at = 0;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            R.c[q] = 0;
            R.v[q] = VT(0);
        }
        if (!own) return;
        const int s = row >> (6 - T.lk);
        const int64_t beg = T.sp[s];
        R.at = (int)beg + ((row << T.lk) & (WAVE - 1));
        R.cnt = (int)((T.sp[s + 1] - beg) >> (6 - T.lk));
        if (R.cnt > 0) fetch(R, 0, R.c, R.v);
    }

    // lane sums of a row (1 << KL of them) and their total as group_sum adds it
    struct Sums {
        AT s[1 << KL];
        __device__ Sums()
        {
#pragma unroll
            for (int q = 0; q < (1 << KL); ++q) s[q] = AT(0);
        }
        __device__ AT total() const
        {
            if constexpr (KL == 0) return s[0];
            else if constexpr (KL == 1) return s[0] + s[1];
            else return (s[0] + s[1]) + (s[2] + s[3]);
        }
    };

    // an exchanged vector (its entries once they are there), or S_l v
    __device__ void gather(const BT *src, const int *c, AT *x) const
    {
        if (!src) {
#pragma unroll
            for (int q = 0; q < U; ++q) x[q] = (AT)(a.v[c[q]] * a.sl[c[q]]);
            return;
        }
        BT b[U];
        unsigned polls = 0;
        for (;;) {
            bool ready = true;
#pragma unroll
            for (int q = 0; q < U; ++q)
                b[q] = __hip_atomic_load(src + c[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int q = 0; q < U; ++q) ready = ready && b[q] != NR;
            if (ready || ++polls > SMALL_WAIT_POLLS) break;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = __builtin_bit_cast(AT, b[q]);
    }

    __device__ void dot(const Row &R, Sums &acc, const BT *src) const
    {
        for (int e = 0; e < R.cnt; e += U) {
            int c[U];
            VT v[U];
            if (e == 0) {
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    c[q] = R.c[q];
                    v[q] = R.v[q];
                }
            } else {
                fetch(R, e, c, v);
            }
            AT x[U];
            gather(src, c, x);
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (e + q < R.cnt) acc.s[q & ((1 << KL) - 1)] += (AT)v[q] * x[q];
        }
    }

    __device__ void run()
    {
        const unsigned turn = a.ep[blockIdx.x];
        BT *set = (BT *)a.ex + (size_t)(turn & 1u) * a.ne * a.n;
        BT *other = (BT *)a.ex + (size_t)(~turn & 1u) * a.ne * a.n;
        Row rL, rU;
        load(rL, a.L);
        load(rU, a.U);
        const AT sv = own ? (AT)(a.v[row] * a.sl[row]) : AT(0);
        const double sr = own ? a.sr[row] : 0.0;
        if (own)
            for (int q = 0; q < a.ne; ++q) other[(size_t)q * a.n + row] = NR;

        // the row's entry of the next exchanged vector, gathered from then on
        const BT *src = nullptr;
        auto put = [&](AT x) {
            BT b = __builtin_bit_cast(BT, x);
            if (b == NR) b ^= BT(1);
            if (own) __hip_atomic_store(set + row, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            src = set;
            set += a.n;
            __asm__ volatile("" ::: "memory");
        };
        const int inner = a.jr ? 0 : a.inner, compact = a.jr ? 0 : a.compact;
        const int per = !a.jr && a.variant == GS2_SYMMETRIC ? 2 : 1, halves = a.sweeps * per;
        const AT w = (AT)a.omega, gamma = (AT)a.gamma;
        const bool damp = !a.jr && a.gamma != 1.0;
        const AT cdiag = compact ? (AT)(1.0 - 1.0 / a.omega) : AT(1);
        bool xzero = true;
        AT x_own = AT(0);
        // x <- w g or x + w g; the last one goes out
        auto finish = [&](bool fin, bool fresh, AT g) {
            x_own = fresh ? w * g : fma(w, g, x_own);
            if (!fin) put(x_own);
            else if (own) a.z[row] = sr * (double)x_own;
        };
        for (int t = 0; t < halves; ++t) {
            const bool lower = a.jr || a.variant == GS2_FORWARD || (a.variant == GS2_SYMMETRIC && t % 2 == 0);
            const bool fin = t == halves - 1, fresh = xzero || compact;
            AT r = sv;
            if (!xzero) {
                Sums acc;
                if (!compact) {
                    if (lower) dot(rL, acc, src);
                    else dot(rU, acc, src);
                }
                if (lower) dot(rU, acc, src);
                else dot(rL, acc, src);
                r = fma(-cdiag, x_own, sv) - acc.total();
            }
            if (inner == 0) {
                finish(fin, fresh, r);
            } else {
                if (!xzero) put(r);
                else src = nullptr; // S_l v
                AT g = r;
                for (int j = 1; j <= inner; ++j) {
                    Sums acc;
                    if (lower) dot(rL, acc, src);
                    else dot(rU, acc, src);
                    const AT old = g;
                    g = fma(-w, acc.total(), r);
                    if (damp) g = fma(gamma, g, (AT(1) - gamma) * old);
                    if (j == inner) finish(fin, fresh, g);
                    else put(g);
                }
            }
            xzero = false;
        }
        if ((threadIdx.x & (WAVE - 1)) == 0) a.ep[blockIdx.x] = turn + 1u;
    }
};

template <typename VT, typename AT, int KL>
__global__ __launch_bounds__(WAVE, 4) void k_small_apply(SmallArgs a)
{
    if (a.stop && *a.stop) return;
    const int row = (int)(blockIdx.x * WAVE + threadIdx.x);
    SmallRow<VT, AT, KL>{a, row, row < a.n}.run();
}

template <typename BT>
__global__ void k_small_reset(int64_t m, BT *__restrict__ ex, BT v, int nw, unsigned *__restrict__ ep)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) ex[i] = v;
    if (i < nw) ep[i] = 0u;
}

template <typename VT, typename AT>
void launch(int lanes, const SmallArgs &a, hipStream_t s)
{
    const unsigned g = (unsigned)((a.n + WAVE - 1) / WAVE);
    if (lanes == 1) k_small_apply<VT, AT, 0><<<g, WAVE, 0, s>>>(a);
    else if (lanes == 2) k_small_apply<VT, AT, 1><<<g, WAVE, 0, s>>>(a);
    else k_small_apply<VT, AT, 2><<<g, WAVE, 0, s>>>(a);
}

ResSell small_view(const Sell &T)
{
    int lk = 0;
    while ((1 << lk) < T.K) ++lk;
    return ResSell{T.slice_ptr, T.col, T.val, lk};
}

} // namespace

int exchanged(bool jr, int sweeps, int inner, int variant)
{
    const int64_t halves = (int64_t)sweeps * (!jr && variant == GS2_SYMMETRIC ? 2 : 1);
    const int64_t passes = jr || inner == 0 ? halves : halves * inner + halves - 1;
    return (int)std::min<int64_t>(passes - 1, 1 << 20);
}

size_t small_bytes(const Handle &h)
{
    const int ne = exchanged(false, h.sweeps, h.inner, h.variant);
    if (h.n > SMALL_MAX_N || h.blocks > 1 || ne < 0 || ne > SMALL_MAX_EX) return 0;
    return aligned(2 * ne * (size_t)h.n * (h.precision == GS2_FP64 ? 8 : 4)) + aligned(4 * ((h.n + WAVE - 1) / WAVE));
}

void small_init(Handle &h, void *mem, hipStream_t s)
{
    h.ne = exchanged(false, h.sweeps, h.inner, h.variant);
    const int64_t m = 2 * h.ne * h.n;
    const int nw = (int)((h.n + WAVE - 1) / WAVE);
    h.ex = mem;
    h.ep = (unsigned *)((char *)mem + small_bytes(h) - aligned(4 * (size_t)nw));
    const unsigned g = (unsigned)((std::max<int64_t>(m, nw) + 255) / 256);
    if (h.precision == GS2_FP64)
        k_small_reset<<<g, 256, 0, s>>>(m, (Bits<double>::T *)mem, Bits<double>::not_ready, nw, h.ep);
    else k_small_reset<<<g, 256, 0, s>>>(m, (Bits<float>::T *)mem, Bits<float>::not_ready, nw, h.ep);
}

bool small_apply(Handle &h, bool jr, int sweeps, double omega, const double *v, double *z, hipStream_t s)
{
    const int lanes = h.fmt == FMT_DIA ? 1 : h.L.K;
    const int ne = exchanged(jr, sweeps, h.inner, h.variant);
    if (!h.ep || ne < 0 || ne > h.ne || lanes > SMALL_LANES || h.fin.st || prof_on()) return false;
    SmallArgs a{};
    a.stop = h.stop;
    a.n = (int)h.n;
    a.ne = h.ne;
    a.jr = jr;
    a.sweeps = sweeps;
    a.inner = h.inner;
    a.variant = h.variant;
    a.compact = h.compact;
    a.omega = omega;
    a.gamma = h.gamma;
    a.L = small_view(h.L);
    a.U = small_view(h.U);
    a.sl = h.sl;
    a.sr = h.sr;
    a.v = v;
    a.z = z;
    a.ex = h.ex;
    a.ep = h.ep;
    if (h.precision == GS2_FP64) launch<double, double>(lanes, a, s);
    else if (h.precision == GS2_FP32) launch<float, float>(lanes, a, s);
    else launch<_Float16, float>(lanes, a, s);
    return true;
}

} // namespace gs2
