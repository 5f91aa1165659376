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
// The wavefronts wait for each other, and nothing makes all of an apply run at
// once: other kernels may hold the compute units that the rest of it needs, for
// seconds or, where they are such applies too, until this one is done.  So a
// wavefront waits for SMALL_WAIT_POLLS looks only.  It then forms what it waits for
// itself, vector by vector and every entry that is not there yet (complete()), and
// starts over with its own rows, which find all they need.  An entry's bits do not
// depend on who forms it, and formed twice it is stored twice alike; a wavefront
// that gets to run only now finds the entries there.  One wavefront alone could do
// the whole apply.
//
// Sums, roundings and therefore every bit are those of the passes launched one
// by one (sweep.hip: Launch::gs2 and Launch::jr), for which fused operations
// are written out where the compiler could fuse another pair.
//
// Enqueued one after the other, SGS2(1,1) in float64 (a call, in us): 11.6
// pass by pass and 6.5 in one launch on 64 x 64 points, 11.9 and 6.8 on 256 x
// 256; GS2(2,2) in float32 19.6 and 7.4, 19.2 and 8.5.  What is left is the
// host's time to enqueue one launch, which the way out of a wait leaves as it was
// (64 x 64 points, 7.0 us a call with it and without).  More rows would gain too, but
// wavefronts that wait for each other should fit next to those of other streams.
#include <algorithm>

#include "gs2_internal.hpp"
#include "resident.hpp"

namespace gs2 {

namespace {

// Looks before a wavefront goes on by itself, half a microsecond or more each
// (counted, not timed: a process that shares the device may be set aside for any
// time): 2 ms, some times what forming the vectors takes where all wavefronts do it at
// once.  With no look allowed an apply (SGS2(1,1) and (1,2), us) takes 41 and 79 on
// 64 x 64 points, 485 and 768 on 256 x 256.
constexpr unsigned SMALL_WAIT_POLLS = 1u << 12;
// In complete() every entry waited for is stored already; a bound all the same.
constexpr unsigned SMALL_STORED_POLLS = 1u << 22;
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
    unsigned looks; // before a wait ends
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
    unsigned looks;
    bool late = false; // a wait has ended without what it waited for

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
    __device__ void gather(const BT *src, const int *c, AT *x)
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
            if (ready || late) break;
            late = ++polls > looks;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = __builtin_bit_cast(AT, b[q]);
    }

    __device__ void dot(const Row &R, Sums &acc, const BT *src)
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

    // what the passes form of a row: the residual S_l v - ... of a half sweep after
    // the first, and the next inner iterate (T: the triangle that the half sweep
    // solves with, O: the other one)
    __device__ AT residual(const Row &T, const Row &O, const BT *src, AT sv, AT x_own)
    {
        const bool compact = !a.jr && a.compact;
        const AT cdiag = compact ? (AT)(1.0 - 1.0 / a.omega) : AT(1);
        Sums acc;
        if (!compact) dot(T, acc, src);
        dot(O, acc, src);
        return fma(-cdiag, x_own, sv) - acc.total();
    }
    __device__ AT relax(const Row &T, const BT *src, AT r, AT old)
    {
        const AT w = (AT)a.omega, gamma = (AT)a.gamma;
        Sums acc;
        dot(T, acc, src);
        AT g = fma(-w, acc.total(), r);
        if (a.gamma != 1.0) g = fma(gamma, g, (AT(1) - gamma) * old);
        return g;
    }
    // x <- w g (fresh: x is zero or replaced) or x + w g
    __device__ AT updated(bool fresh, AT x_own, AT g) const
    {
        const AT w = (AT)a.omega;
        return fresh ? w * g : fma(w, g, x_own);
    }
    __device__ AT scaled_v() const { return own ? (AT)(a.v[row] * a.sl[row]) : AT(0); }
    __device__ void store(BT *vec, AT x) const
    {
        BT b = __builtin_bit_cast(BT, x);
        if (b == NR) b ^= BT(1);
        if (own) __hip_atomic_store(vec + row, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ BT fetched(const BT *vec) const
    {
        return own ? __hip_atomic_load(vec + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : BT(0);
    }

    // half sweeps, and whether one solves with the lower triangle
    __device__ static int halves(const SmallArgs &a) { return a.sweeps * (!a.jr && a.variant == GS2_SYMMETRIC ? 2 : 1); }
    __device__ static bool lower_half(const SmallArgs &a, int t)
    {
        return a.jr || a.variant == GS2_FORWARD || (a.variant == GS2_SYMMETRIC && t % 2 == 0);
    }

    // the row through all passes; false (in every lane) once a wait has ended
    __device__ bool run(BT *set, BT *other, unsigned limit)
    {
        looks = limit;
        late = false;
        Row rL, rU;
        load(rL, a.L);
        load(rU, a.U);
        const AT sv = scaled_v();
        const double sr = own ? a.sr[row] : 0.0;
        if (own)
            for (int q = 0; q < a.ne; ++q) other[(size_t)q * a.n + row] = NR;

        // the row's entry of the next exchanged vector, gathered from then on
        const BT *src = nullptr;
        auto put = [&](AT x) {
            store(set, x);
            src = set;
            set += a.n;
            __asm__ volatile("" ::: "memory");
        };
        const int inner = a.jr ? 0 : a.inner, H = halves(a);
        AT x_own = AT(0);
        auto finish = [&](bool fin, bool fresh, AT g) {
            x_own = updated(fresh, x_own, g);
            if (!fin) put(x_own);
            else if (own) a.z[row] = sr * (double)x_own;
        };
        for (int t = 0; t < H; ++t) {
            const bool lower = lower_half(a, t), fin = t == H - 1, fresh = t == 0 || (!a.jr && a.compact);
            AT r = sv;
            if (t > 0) {
                r = lower ? residual(rL, rU, src, sv, x_own) : residual(rU, rL, src, sv, x_own);
                if (__any(late)) return false;
            }
            if (inner == 0) {
                finish(fin, fresh, r);
                continue;
            }
            if (t > 0) put(r);
            else src = nullptr; // S_l v
            AT g = r;
            for (int j = 1; j <= inner; ++j) {
                g = lower ? relax(rL, src, r, g) : relax(rU, src, r, g);
                if (__any(late)) return false;
                if (j == inner) finish(fin, fresh, g);
                else put(g);
            }
        }
        return true;
    }

    // Every entry of the apply's exchanged vectors that is not there yet, one vector
    // after the other (each needs all of the one before it and, of its own row, the
    // half sweep's residual and the iterate before it).  The wavefront starts with its
    // own rows, as others that do the same start with theirs.
    __device__ static void complete(const SmallArgs &a, BT *set)
    {
        const int inner = a.jr ? 0 : a.inner, H = halves(a), nc = (a.n + WAVE - 1) / WAVE;
        const BT *x = nullptr, *r = nullptr, *src = nullptr; // iterate, residual, the vector before
        for (int t = 0; t < H; ++t) {
            const bool lower = lower_half(a, t), fresh = t == 0 || (!a.jr && a.compact);
            r = nullptr;
            // pass 0: the residual (itself, or the iterate it gives); j > 0: inner pass j
            for (int pass = t == 0 && inner > 0 ? 1 : 0; pass <= inner; ++pass) {
                const bool last = pass == inner;
                if (last && t == H - 1) return; // the output
                for (int k = 0; k < nc; ++k) {
                    const int c = ((int)blockIdx.x + k) % nc, row = c * WAVE + (int)(threadIdx.x & (WAVE - 1));
                    SmallRow w{a, row, row < a.n, SMALL_STORED_POLLS};
                    if (!__any(w.own && w.fetched(set) == NR)) continue;
                    Row T, O;
                    w.load(T, lower ? a.L : a.U);
                    w.load(O, lower ? a.U : a.L);
                    const AT sv = w.scaled_v();
                    const AT xo = x ? __builtin_bit_cast(AT, w.fetched(x)) : AT(0);
                    AT g;
                    if (pass == 0) {
                        g = t == 0 ? sv : w.residual(T, O, src, sv, xo);
                    } else {
                        const AT rr = r ? __builtin_bit_cast(AT, w.fetched(r)) : sv;
                        g = w.relax(T, src, rr, pass == 1 ? rr : __builtin_bit_cast(AT, w.fetched(src)));
                    }
                    w.store(set, last ? w.updated(fresh, xo, g) : g);
                }
                src = set;
                if (last) x = set;
                else if (pass == 0) r = set;
                set += a.n;
            }
        }
    }
};

// The kernel's arguments, read again where the call stands: the way that is hardly
// ever taken then keeps nothing in scalar registers, which spilled, on the other.
__device__ __forceinline__ SmallArgs arguments()
{
    static_assert(sizeof(SmallArgs) % 4 == 0, "whole words");
    auto p = (const __attribute__((address_space(4))) unsigned *)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(p));
    unsigned w[sizeof(SmallArgs) / 4];
#pragma unroll
    for (unsigned k = 0; k < sizeof(SmallArgs) / 4; ++k) w[k] = p[k];
    SmallArgs a;
    __builtin_memcpy(&a, w, sizeof a);
    return a;
}

template <typename VT, typename AT, int KL>
__global__ __launch_bounds__(WAVE, 4) void k_small_apply(SmallArgs a)
{
    if (a.stop && *a.stop) return;
    using R = SmallRow<VT, AT, KL>;
    using BT = typename R::BT;
    const int row = (int)(blockIdx.x * WAVE + threadIdx.x);
    const unsigned turn = a.ep[blockIdx.x];
    BT *set = (BT *)a.ex + (size_t)(turn & 1u) * a.ne * a.n;
    BT *other = (BT *)a.ex + (size_t)(~turn & 1u) * a.ne * a.n;
    if (!R{a, row, row < a.n}.run(set, other, a.looks)) {
        R::complete(arguments(), set);
        const SmallArgs b = arguments();
        (void)R{b, row, row < b.n}.run(set, other, SMALL_STORED_POLLS);
    }
    if (threadIdx.x == 0) a.ep[blockIdx.x] = turn + 1u;
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

bool small_suits(const Handle &h, const Pattern &pat)
{
    if (pat.maxlen > SMALL_MAX_ROW) return false;
    const bool scattered = pat.many_d && pat.nl + pat.nu >= 3 * h.n;
    return !scattered || pat.far <= (h.precision == GS2_FP64 ? SMALL_FAR_64 : SMALL_FAR_32);
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
    // a single Jacobi sweep gathers nothing and is one launch as it is (7.4 us, 7.8 here)
    if ((jr || h.inner == 0) && sweeps == 1 && (jr || h.variant != GS2_SYMMETRIC)) return false;
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
    a.looks = h.wait_looks < 0 ? SMALL_WAIT_POLLS : (unsigned)h.wait_looks;
    if (h.precision == GS2_FP64) launch<double, double>(lanes, a, s);
    else if (h.precision == GS2_FP32) launch<float, float>(lanes, a, s);
    else launch<_Float16, float>(lanes, a, s);
    ++h.one_launch_applies;
    return true;
}

} // namespace gs2

extern "C" int gs2_wait_looks(gs2_handle *H, int looks)
{
    if (!H) return GS2_ERR_ARG;
    H->h.wait_looks = looks;
    return GS2_OK;
}

extern "C" int gs2_paths(const gs2_handle *H, int *last_solve, int *paired, int64_t *given_up, int64_t *applies,
                         int *timings)
{
    if (!H) return GS2_ERR_ARG;
    if (last_solve) *last_solve = H->h.last_solve;
    if (paired) *paired = H->h.paired;
    if (given_up) *given_up = H->h.given_up;
    if (applies) *applies = H->h.one_launch_applies;
    if (timings) *timings = gs2::timings(H->h.gw);
    return GS2_OK;
}
