// A whole GMRES solve of a small system in one launch.
//
// Below some ten thousand rows a restart cycle launched kernel by kernel (or
// replayed from a graph) is a chain of launches: six to ten per Arnoldi step
// at 4 to 5 us each, whatever they do, and the launches of a cycle that are
// left over once it has converged.  Here G workgroups stay for the whole
// solve, each with its own contiguous rows, and meet at a barrier between
// cycles (0.8 us for up to 32 of them, 1.3 us for 64).  64 x 64 Poisson,
// SGS2(1,1), GMRES(30), 92 steps: 3.17 ms launched, 1.26 ms here; 255 x 255
// convection-diffusion, GS2(2,2), GMRES(20), 114 steps: 6.39 against 3.07 ms.
// (With a barrier after every pass, 0.8 to 1.3 us and the stores' acknowledgement
// before it, 1.99 and 4.88 ms.)  Bound by the chain of trips past the caches: one
// for every pass of the preconditioner, for the product and for either
// reduction of a step, about 0.8 us each, and by the serial work of a step
// (3.5 us, on a wavefront of its own where 1024 threads leave room for one).
//
// Rows per workgroup: the fewest that 64 workgroups hold (64 partial sums are
// one per lane).  64 x 64 Poisson with 1024 rows per workgroup and barriers took
// 2.19 ms, with 256 and barriers 1.99.
//
// Method, order of every sum and therefore every bit are those of krylov.hip's
// delayed reorthogonalisation launch by launch: a workgroup here owns the
// rows that a workgroup of the launches owns (res_rows), forms its partial sums in
// the same order and adds the partials of all workgroups as k_reduce and
// dcgs_finish_block do (at most 64 of them: one per lane).  Every workgroup
// does so, repeats the scalar work on its own copy of the state
// (dcgs_state.hpp) and takes the same branches.
//
// Memory: what other workgroups read (the vectors that a pass gathers, partial
// sums) is only ever stored and loaded at agent scope, past the caches that
// XCDs do not share; what only its own workgroup reads (the basis V, the
// preconditioned vectors Z) is only ever accessed plainly.  The matrix is read
// plainly and never written.
//
// Within a cycle there is no barrier between workgroups: an entry of an
// exchanged vector and a partial sum is its own flag (Bits::not_ready until it
// is there) and readers poll, one trip instead of the four of store, arrival,
// departure and load.  A step uses one of two turns of the exchanged vectors and
// one of three turns of the partial sums.  A workgroup that has seen every
// first-pass sum of step j knows that all are done with the vectors of step j
// and the sums of step j - 1, and resets its own entries of these; it waits for
// the resets to be acknowledged before it publishes its sums of step j + 1,
// without which nobody reads that turn again.  A cycle starts with all of it
// reset, then a barrier.
//
// Registers: 1024 threads leave 128 per thread.  Kept below that without spills
// of vector registers (eight loads in flight over a basis vector, not all sixteen;
// two entries of a row at a time).  The build fails on such a spill here: a version
// that spilled 55 of them beside 139 scalar ones gave wrong results in the float32
// instantiation, the same ones in every run, and the cause was not found (scalar
// registers alone, which go to lanes of vector registers, do no harm).
//
// Waits are bounded: past WAIT_TICKS of the wall clock or ResArgs::looks the
// abort flag goes up, who has waited that long waits no more, every workgroup
// leaves at the next barrier and the caller solves by launches instead, from
// the x it finds (x is written after a barrier past which nothing is waited for).
#include <algorithm>
#include <cmath>

#include "dcgs_state.hpp"
#include "gs2_internal.hpp"
#include "resident.hpp"
#include "sella.hpp"

namespace gs2 {

namespace {

constexpr long long WAIT_TICKS = 200000000ll; // 2 s at 100 MHz
constexpr int QW = KT / WAVE;   // wavefronts of the launches whose sums are repeated here

// Threads of a workgroup of RR rows: one per row and, where there is room for
// it, a wavefront that closes a step while the others precondition.
constexpr int threads_of(int rr) { return rr < 1024 ? rr + WAVE : rr; }
constexpr int near_of(int rr) { return rr < 1024 ? 1 : rr; }

__device__ __forceinline__ double ald(const double *p)
{
    return __longlong_as_double((long long)__hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ float ald(const float *p)
{
    return __uint_as_float(__hip_atomic_load((const unsigned *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void ast(double *p, double v)
{
    __hip_atomic_store((unsigned long long *)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ast(float *p, float v)
{
    __hip_atomic_store((unsigned *)p, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int RR>
struct Shared {
    unsigned long long sw[GSTATE_SMALL_WORDS];
    double col[MAXM + 2], sc[2], red[QW], nrm[3 * QW];
    double step[3]; // alpha, e, alpha^2 of the step to be closed
    double ul[RR], wl[RR];
    // own rows of the vector gathered now, and of the next one, for 1024 rows:
    // read at agent scope every one of them was a trip past the caches
    double near[2][near_of(RR)];
    int flag, most[3];
    unsigned looks; // ResArgs::looks (in a scalar register the polls were 1 % slower)
};

// A stored matrix and a thread's row of it: entry k at col[p], val[p] with
// p = at + (k >> lk) step + (k mod 2^lk), in global memory (sliced ELL) or in
// the workgroup's copy in LDS (entry k of all its rows side by side).
struct Mat {
    const int32_t *col;
    const void *val;
    int lk, step; // the same in every thread
    int at, cnt;
};

// One workgroup's view of the solve.  KL: log2 of the lanes per row whose sums
// the launches add (0 where they add a row's entries one after the other).
template <typename VT, typename AT, int KL, int RR>
struct Team {
    static constexpr int NT = threads_of(RR), NW = NT / WAVE;
    const ResArgs &a;
    Shared<RR> &sh;
    double *H; // m x m, in LDS
    int me, t, wv, ln;
    int r0, rows, row; // the workgroup's first row and row count, the thread's row
    bool own;          // the thread has one
    Mat mL, mU, mA;
    AT sv_own = AT(0); // S_l u, rounded (u itself, unscaled, in sh.ul)
    unsigned epoch = 0;

    static constexpr bool NEAR = near_of(RR) == RR;
    int side = 0; // which of sh.near is gathered
    bool late = false; // a wait has run out
    int turn = 0; // of the exchanged vectors

    __device__ GState *st() const { return reinterpret_cast<GState *>(sh.sw); }

    template <typename T>
    __device__ static void astf(T *p, T v) // an entry that is its own flag
    {
        typename Bits<T>::T b = __builtin_bit_cast(typename Bits<T>::T, v);
        if (b == Bits<T>::not_ready) b ^= 1;
        ast(p, __builtin_bit_cast(T, b));
    }
    template <typename T>
    __device__ static void reset(T *p)
    {
        ast(p, __builtin_bit_cast(T, Bits<T>::not_ready));
    }
    template <typename T>
    __device__ static bool there(T v)
    {
        return __builtin_bit_cast(typename Bits<T>::T, v) != Bits<T>::not_ready;
    }

    // between two looks at entries that are not there yet; false: wait no more
    __device__ bool wait(unsigned &polls)
    {
        if (late) return false;
        if (++polls < sh.looks) return true;
        late = true;
        __hip_atomic_store(a.bar + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }

    // the thread's entry of the vector that the next pass gathers
    template <typename T>
    __device__ void put(T *vec, T v)
    {
        astf(vec + row, v);
        if (NEAR) reinterpret_cast<T *>(sh.near[side ^ 1])[t] = v;
    }
    // what the workgroup's threads have put is gathered from here on
    __device__ void flip()
    {
        side ^= 1;
        if (NEAR) __syncthreads();
        __asm__ volatile("" ::: "memory");
    }

    // U entries of the vector put last: own rows from LDS where they are kept
    // there (most of a mesh row's), others from memory as soon as they are there
    template <int U, typename T>
    __device__ void gather(const T *vec, const int *c, T *x)
    {
        const T *near = reinterpret_cast<const T *>(sh.near[side]);
        unsigned polls = 0;
        for (;;) {
            bool ready = true;
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const unsigned i = (unsigned)(c[q] - r0);
                if (NEAR && i < (unsigned)rows) x[q] = near[i];
                else x[q] = ald(vec + c[q]);
            }
#pragma unroll
            for (int q = 0; q < U; ++q) ready = ready && (there(x[q]) || (NEAR && (unsigned)(c[q] - r0) < (unsigned)rows));
            if (ready || !wait(polls)) return;
        }
    }

    // every workgroup's agent stores before it are seen by every workgroup's
    // agent loads after it; false once the solve has been given up
    __device__ bool meet()
    {
        side ^= 1;
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (a.G == 1) { // a wait may have run out all the same
            if (t == 0) sh.flag = (int)__hip_atomic_load(a.bar + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            return sh.flag == 0;
        }
        ++epoch;
        if (t == 0) {
            sh.flag = 0;
            __hip_atomic_fetch_add(a.bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned target = (unsigned)a.G * epoch;
            const long long t0 = wall_clock64();
            unsigned polls = 0;
            while (__hip_atomic_load(a.bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                if ((++polls & 255u) == 0u) {
                    if (wall_clock64() - t0 > WAIT_TICKS)
                        __hip_atomic_store(a.bar + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (__hip_atomic_load(a.bar + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
                }
            }
            if (__hip_atomic_load(a.bar + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) sh.flag = 1;
        }
        __syncthreads();
        __asm__ volatile("" ::: "memory");
        return sh.flag == 0;
    }

    // A lane's sums of a row (1 << KL of them) and their total as group_sum adds it.
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

    __device__ Mat row_of(const ResSell &T) const
    {
        if (!own) return Mat{T.col, T.val, T.lk, WAVE, 0, 0};
        const int s = row >> (6 - T.lk);
        const int64_t beg = T.sp[s];
        return Mat{T.col, T.val, T.lk, WAVE, (int)beg + ((row << T.lk) & (WAVE - 1)),
                   (int)((T.sp[s + 1] - beg) >> (6 - T.lk))};
    }

    // move the rows' entries into LDS, `used` bytes into the area `area`, if
    // they fit
    template <typename WT>
    __device__ void keep(Mat &M, int which, char *area, int &used, int size)
    {
        atomicMax(&sh.most[which], M.cnt);
        __syncthreads();
        const int most = __builtin_amdgcn_readfirstlane(sh.most[which]);
        const int bytes = most * RR * (int)(sizeof(WT) + sizeof(int32_t));
        if (used + bytes > size) return;
        WT *val = (WT *)(area + used);
        int32_t *col = (int32_t *)(val + most * RR);
        for (int k = 0; k < M.cnt; ++k) {
            const int p = M.at + (k >> M.lk) * M.step + (k & ((1 << M.lk) - 1));
            val[k * RR + t] = ((const WT *)M.val)[p];
            col[k * RR + t] = M.col[p];
        }
        M.val = val;
        M.col = col;
        M.lk = 0;
        M.step = RR;
        M.at = t;
        used += bytes;
    }

    // f(values, columns, entries left) over the row's stored entries, U at a time
    template <typename WT, int U, typename F>
    __device__ void each_entry(const Mat &M, F f) const
    {
        const WT *val = (const WT *)M.val;
        const int km = (1 << M.lk) - 1;
        for (int e = 0; e < M.cnt; e += U) {
            int c[U];
            WT v[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int k = e + q < M.cnt ? e + q : M.cnt - 1;
                const int p = M.at + (k >> M.lk) * M.step + (k & km);
                c[q] = M.col[p];
                v[q] = val[p];
            }
            f(v, c, M.cnt - e);
        }
    }

    // acc += the row's stored entries of T times vec at their columns
    __device__ void row_dot(const Mat &T, Sums &acc, const AT *vec)
    {
        constexpr int U = NEAR && KL < 2 ? 2 : 4; // what the registers hold
        each_entry<VT, U>(T, [&](const VT *v, const int *c, int left) {
            AT x[U];
            gather<U>(vec, c, x);
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (q < left) acc.s[q & ((1 << KL) - 1)] += (AT)v[q] * x[q];
        });
    }

    // (A x)[row] in float64
    __device__ double a_row(const double *vec)
    {
        double acc = 0.0;
        constexpr int U = !NEAR && KL == 0 ? 8 : 4; // a 7-point row in one round trip, where the registers last
        each_entry<double, U>(mA, [&](const double *v, const int *c, int left) {
            double x[U];
            gather<U>(vec, c, x);
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (q < left) acc += v[q] * x[q];
        });
        return acc;
    }

    // the vectors of a turn: S_l u and the preconditioner's, z
    __device__ AT *ex(int tn, int q) const { return (AT *)a.ex + (int64_t)(tn * (a.ne + 1) + q) * a.n; }
    __device__ double *ze(int tn) const { return a.ze + (int64_t)tn * a.n; }

    // z_j into the plain column (read back by this thread) and the gathered vector
    __device__ void put_z(double *zcol, double z)
    {
        zcol[row] = z;
        put(ze(turn), z);
    }

    // the next raw tentative vector: the thread's entry, and S_l u for the
    // preconditioner's gathers (rounded as the launches round it)
    __device__ void put_u(double u, int tn)
    {
        sh.ul[t] = u;
        if (a.kind == GS2_PREC_NONE) return;
        sv_own = (AT)(u * a.sl[row]);
        put(ex(tn, 0), sv_own);
    }

    // z = Mhat^{-1} u on the raw tentative vector (Launch::gs2 and Launch::jr of
    // sweep.hip, pass by pass).  What a pass needs of the thread's own row it
    // still holds; only other rows' entries are gathered.
    __device__ void precondition(double *zcol)
    {
        if (a.kind == GS2_PREC_NONE) {
            if (own) put_z(zcol, sh.ul[t]);
            flip();
            return;
        }
        const bool jr = a.kind == GS2_PREC_JR;
        const int inner = jr ? 0 : a.inner, compact = jr ? 0 : a.compact;
        const int per = !jr && a.variant == GS2_SYMMETRIC ? 2 : 1, Hh = a.sweeps * per;
        const AT w = (AT)a.omega, gamma = (AT)a.gamma;
        const bool damp = a.gamma != 1.0 && !jr;
        const AT cdiag = compact ? (AT)(1.0 - 1.0 / a.omega) : AT(1);
        bool xzero = true;
        AT x_own = AT(0);
        AT *src = ex(turn, 0); // the vector gathered
        int used = 0;
        // the row's entry of the next one
        auto next = [&](AT v) {
            ++used;
            if (own) put(ex(turn, used), v);
            src = ex(turn, used);
            flip();
        };
        // x <- w g or x + w g, or the output
        auto finish = [&](bool fin, bool set, AT g) {
            const AT x = set ? w * g : fma(w, g, x_own);
            x_own = x;
            if (!fin) {
                next(x);
                return;
            }
            if (own) put_z(zcol, a.sr[row] * (double)x);
            flip();
        };
        for (int tt = 0; tt < Hh; ++tt) {
            const bool lower = jr || a.variant == GS2_FORWARD || (a.variant == GS2_SYMMETRIC && tt % 2 == 0);
            const Mat &T = lower ? mL : mU, &O = lower ? mU : mL;
            const bool fin = tt == Hh - 1, set = xzero || compact;
            AT r = sv_own;
            if (!xzero) {
                Sums acc;
                if (!compact) row_dot(T, acc, src);
                row_dot(O, acc, src);
                r = fma(-cdiag, x_own, sv_own) - acc.total();
            }
            if (inner == 0) {
                finish(fin, set, r);
            } else {
                if (!xzero) next(r);
                AT g = r;
                for (int j = 1; j <= inner; ++j) {
                    Sums acc;
                    row_dot(T, acc, src);
                    const AT old = g;
                    g = fma(-w, acc.total(), r);
                    if (damp) g = fma(gamma, g, (AT(1) - gamma) * old);
                    if (j == inner) finish(fin, set, g);
                    else next(g);
                }
            }
            xzero = false;
        }
    }

    // sums of the workgroups' partials part[q * G ..), one per lane, for q = q0,
    // q0 + dq, .. (one wavefront; every lane gets them), PF polled at a time
    template <int PF>
    __device__ void totals(const double *part, int q0, int dq, int last, double *o)
    {
        unsigned polls = 0;
        for (;;) {
            bool ready = true;
#pragma unroll
            for (int p = 0; p < PF; ++p) o[p] = ln < a.G ? ald(part + min(q0 + p * dq, last) * a.G + ln) : 0.0;
#pragma unroll
            for (int p = 0; p < PF; ++p) ready = ready && there(o[p]);
            if (ready || !wait(polls)) break;
        }
#pragma unroll
        for (int p = 0; p < PF; ++p) o[p] = wave_sum(o[p]);
    }
    __device__ double total(const double *part)
    {
        double o[1];
        totals<1>(part, 0, 0, 0, o);
        return o[0];
    }

    // the workgroup's sum of squares of one value per row (0 without a row):
    // a thread of KT adds its rows t, t + KT, ..., then block_sum; to part[me]
    __device__ void publish_squares(double v, double *part)
    {
        if (NT == RR || t < RR) sh.wl[t] = v;
        __syncthreads();
        if (t < KT) {
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < RR / KT; ++u) s = fma(sh.wl[t + u * KT], sh.wl[t + u * KT], s);
            s = wave_sum(s);
            if (ln == 0) sh.red[wv] = s;
        }
        __syncthreads();
        if (t == 0) {
            double s = 0.0;
            for (int k = 0; k < QW; ++k) s += sh.red[k];
            astf(part + me, s);
        }
    }

    // the total of the published sums, in every thread
    __device__ double agree(const double *part)
    {
        if (wv == 0) {
            const double s = total(part);
            if (ln == 0) sh.sc[0] = s;
        }
        __syncthreads();
        const double s = sh.sc[0];
        __syncthreads();
        return s;
    }

    __device__ bool solve(ResInfo &info);
};

template <typename VT, typename AT, int KL, int RR>
__device__ bool Team<VT, AT, KL, RR>::solve(ResInfo &info)
{
    GState *ls = st();
    const int n = a.n, m = a.m;
    // a norm between barriers; a step's norm and first-pass sums, three turns
    double *const partB = a.part;
    const int turn_size = a.G * (2 * m + 4);
    auto partN = [&](int j) { return a.part + a.G + (j % 3) * turn_size; };
    auto partQ = [&](int j) { return partN(j) + a.G; };
    info = ResInfo{0, 0, GS2_OK, 0, 0.0};
    // the rows into LDS, the triangles first: they are read most often
    {
        char *area = (char *)(H + m * m);
        const int size = a.lds - (int)sizeof(double) * m * m;
        int used = 0;
        mL = row_of(a.L);
        mU = row_of(a.U);
        mA = row_of(a.A);
        if (t < 3) sh.most[t] = 0;
        if (t == 0) sh.looks = a.looks;
        __syncthreads();
        if (a.kind != GS2_PREC_NONE) {
            keep<VT>(mL, 0, area, used, size);
            keep<VT>(mU, 1, area, used, size);
        }
        keep<double>(mA, 2, area, used, size);
    }
    if (own) put(a.xe, a.x[row]);
    publish_squares(own ? a.b[row] : 0.0, partB);
    if (!meet()) return false;
    const double bnorm = sqrt(agree(partB));
    if (!isfinite(bnorm)) {
        info.status = GS2_ERR_NONFINITE;
        return true;
    }
    if (bnorm == 0.0) {
        if (own) a.x[row] = 0.0;
        info.converged = 1;
        return true;
    }
    double ref_res = -1.0;
    int cycles = 0, ref_cycle = 0;
    for (;;) {
        // true residual
        const double r = own ? a.b[row] - a_row(a.xe) : 0.0;
        if (!meet()) return false; // the norms read last are no longer needed
        publish_squares(r, partB);
        if (!meet()) return false;
        const double beta = sqrt(agree(partB));
        if (cycles > 0) {
            info.iterations += ls->kk;
            if (ls->status != GS2_OK) {
                info.status = ls->status;
                break;
            }
        }
        info.relres = beta / bnorm;
        if (!isfinite(beta)) {
            info.status = GS2_ERR_NONFINITE;
            break;
        }
        if (info.relres <= a.rtol) {
            info.converged = 1;
            break;
        }
        if (info.iterations >= a.maxit) {
            info.status = GS2_NOT_CONVERGED;
            break;
        }
        if (ref_res < 0.0 || info.relres < 0.5 * ref_res) {
            ref_res = info.relres;
            ref_cycle = cycles;
        } else if (a.stag > 0 && cycles - ref_cycle >= a.stag) {
            info.status = GS2_STAGNATED;
            break;
        }
        if (cycles > 0) info.restarts++;
        ++cycles;
        const int steps = min(m, a.maxit - info.iterations);
        // a new cycle: state, and the normalised residual as the first vector
        __syncthreads();
        for (int k = t; k < GSTATE_SMALL_WORDS; k += NT) sh.sw[k] = 0ull;
        __syncthreads();
        for (int k = t; k < MAXM + 2; k += NT) ls->zs[k] = 1.0;
        if (t == 0) {
            ls->status = GS2_OK;
            ls->maxsteps = steps;
            ls->rtol = a.rtol;
            ls->bnorm = bnorm;
            ls->beta = beta;
            ls->g[0] = beta;
        }
        if (own)
            for (int tn = 0; tn < 2; ++tn) {
                for (int q = 0; q <= a.ne; ++q) reset(ex(tn, q) + row);
                reset(ze(tn) + row);
            }
        for (int k = t; k < 3 * (2 * m + 4); k += NT) reset(a.part + a.G + k * a.G + me);
        if (!meet()) return false;
        if (own) put_u(r * (1.0 / beta), 0);
        flip();
        bool ok = true;
        for (int j = 0;; ++j) {
            // the serial work that closes step j - 1, on one wavefront; unless
            // it ends the cycle for sure, beside the other wavefronts' share
            // of the next preconditioner's first pass, which needs neither the
            // scale nor the test it forms
            if (j > 0) {
                if (wv == NW - 1)
                    dcgs_finish_wave(ls, H, m, sh.col, ok, sh.step[0], sh.step[1], sh.step[2],
                                     ok ? total(partN(j - 1)) : 0.0);
                if (j == steps || !ok) {
                    __syncthreads();
                    break;
                }
            }
            turn = j & 1;
            if (NW * WAVE == RR || wv != NW - 1) precondition(a.Z + (int64_t)j * n);
            __syncthreads();
            if (ls->done) break;
            // w = A z_j and u, scaled
            const double zsc = ls->zs[j];
            const double ws = own ? zsc * a_row(ze(turn)) : 0.0;
            if (NT == RR || t < RR) {
                sh.wl[t] = ws;
                sh.ul[t] = own ? zsc * sh.ul[t] : 0.0;
            }
            __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); // the resets, before anything is published
            __syncthreads();
            double *const pq = partQ(j);
            // a = Q^T u, c = Q^T w, a column per wavefront in turn; the first
            // QW of them start with u.u, u.w, w.w (as block_multidot)
            if (wv < QW) {
                double aa = 0.0, ab = 0.0, bb = 0.0;
#pragma unroll
                for (int q = 0; q < RR / KT; ++q) {
                    const double x = sh.ul[ln + (wv * (RR / KT) + q) * WAVE];
                    const double y = sh.wl[ln + (wv * (RR / KT) + q) * WAVE];
                    aa = fma(x, x, aa);
                    ab = fma(x, y, ab);
                    bb = fma(y, y, bb);
                }
                aa = wave_sum(aa);
                ab = wave_sum(ab);
                bb = wave_sum(bb);
                if (ln == 0) {
                    sh.nrm[3 * wv] = aa;
                    sh.nrm[3 * wv + 1] = ab;
                    sh.nrm[3 * wv + 2] = bb;
                }
            }
            for (int k = NW - 1 - wv; k < j; k += NW) {
                const double *__restrict__ vk = a.V + (int64_t)k * n + r0;
                double sa = 0.0, sb = 0.0;
                constexpr int U = std::min(RR / WAVE, 8); // loads in flight
#pragma unroll 1
                for (int q0 = 0; q0 < RR / WAVE; q0 += U) {
                    double x[U];
#pragma unroll
                    for (int q = 0; q < U; ++q) x[q] = vk[min(ln + (q0 + q) * WAVE, rows - 1)];
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        sa += x[q] * sh.ul[ln + (q0 + q) * WAVE];
                        sb += x[q] * sh.wl[ln + (q0 + q) * WAVE];
                    }
                }
                sa = wave_sum(sa);
                sb = wave_sum(sb);
                if (ln == 0) {
                    astf(pq + k * a.G + me, sa);
                    astf(pq + (j + k) * a.G + me, sb);
                }
            }
            __syncthreads();
            if (t < 3) {
                double o = 0.0;
                for (int q = 0; q < QW; ++q) o += sh.nrm[3 * q + t];
                astf(pq + (2 * j + t) * a.G + me, o);
            }
            constexpr int PF = RR < 512 ? 8 : 4; // loads in flight
            for (int q0 = wv; q0 < 2 * j + 3; q0 += PF * NW) {
                double o[PF];
                totals<PF>(pq, q0, NW, 2 * j + 2, o);
#pragma unroll
                for (int p = 0; p < PF; ++p) {
                    const int q = q0 + p * NW;
                    const double v = o[p];
                    if (ln == 0 && q < 2 * j + 3) {
                        if (q < j) ls->hA[q] = v;
                        else if (q < 2 * j) ls->hB[q - j] = v;
                        else if (q == 2 * j) ls->bb = v;
                        else if (q == 2 * j + 1) ls->dd = v;
                        else ls->wn2 = v;
                    }
                }
            }
            __syncthreads();
            // nobody needs the vectors of this step and the sums of the last one any more
            if (own) {
                for (int q = 0; q <= a.ne; ++q) reset(ex(turn, q) + row);
                reset(ze(turn) + row);
            }
            for (int k = t; k < 2 * m + 4; k += NT) reset(partN(j + 2) + k * a.G + me);
            double alpha, e, a2;
            ok = reorth_scalars(ls, j, ls->hA, ls->hB, sh.sc, &alpha, &e, &a2);
            if (wv == NW - 1 && ln == 0) {
                sh.step[0] = alpha;
                sh.step[1] = e;
                sh.step[2] = a2;
            }
            if (!ok) continue; // u fell into span(Q): the cycle ends on the tentative column j - 1
            // q_j = (u - Q a) / alpha, w' = w - Q c - e q_j
            double wp = 0.0;
            if (own) {
                double aq = sh.ul[t], aw = sh.wl[t]; // rounded products, as the launches read them
                const double *__restrict__ vr = a.V + row;
                constexpr int U = RR < 1024 ? 16 : 4; // loads in flight
                for (int k = 0; k < j; k += U) {
                    double x[U];
#pragma unroll
                    for (int q = 0; q < U; ++q) x[q] = vr[(int64_t)min(k + q, j - 1) * n];
#pragma unroll
                    for (int q = 0; q < U; ++q)
                        if (k + q < j) {
                            aq -= ls->hA[k + q] * x[q];
                            aw -= ls->hB[k + q] * x[q];
                        }
                }
                const double qv = aq * (1.0 / alpha);
                wp = aw - e * qv;
                a.V[(int64_t)j * n + row] = qv;
                put_u(wp, turn ^ 1);
            }
            flip();
            publish_squares(wp, partN(j));
        }
        __syncthreads();
        // y = R^{-1} g (as k_backsolve), x += Z y
        const int kk = ls->kk;
        if (wv == 0) {
            for (int k = kk - 1; k >= 0; --k) {
                double p = 0.0;
                for (int l = k + 1 + ln; l < kk; l += WAVE) p += H[k * m + l] * ls->y[l];
                p = wave_sum(p);
                if (ln == 0) ls->y[k] = (ls->g[k] - p) / H[k * m + k];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // its LDS write before its next reads
            }
        }
        __syncthreads();
        if (own) {
            double xv = ald(a.xe + row);
#pragma unroll 8
            for (int k = 0; k < kk; ++k) xv += (ls->y[k] * ls->zs[k]) * a.Z[(int64_t)k * n + row];
            put(a.xe, xv);
        }
        if (!meet()) return false;
    }
    if (own) a.x[row] = ald(a.xe + row);
    return true;
}

template <typename VT, typename AT, int KL, int RR>
__global__ __launch_bounds__(threads_of(RR)) void k_resident(ResArgs a)
{
    extern __shared__ double hl[];
    __shared__ Shared<RR> sh;
    const int t = threadIdx.x, r0 = (int)blockIdx.x * RR, rows = min(RR, a.n - r0);
    Team<VT, AT, KL, RR> T{a, sh, hl, (int)blockIdx.x, t, __builtin_amdgcn_readfirstlane(t / WAVE), t & (WAVE - 1), r0, rows, r0 + t,
                           t < rows, Mat{}, Mat{}, Mat{}};
    ResInfo info;
    const bool done = T.solve(info);
    if (t == 0) {
        if (blockIdx.x == 0) *a.info = info;
        __threadfence_system();
        // the last workgroup to leave marks a solve that any of them gave up
        // and clears the barrier for the next one
        if (__hip_atomic_fetch_add(a.bar + 2, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)a.G - 1u) {
            if (!done || __hip_atomic_load(a.bar + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                a.info->status = RES_GIVEN_UP;
            for (int k = 0; k < 3; ++k)
                __hip_atomic_store(a.bar + k, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <typename VT, typename AT, int KL, int RR>
int launch_rows(ResArgs a, hipStream_t s)
{
    // the Hessenberg matrix and as much of the rows as fits
    int dev = 0, most = 0;
    GS2_TRY_HIP(hipGetDevice(&dev));
    GS2_TRY_HIP(hipDeviceGetAttribute(&most, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    a.lds = std::max((int)sizeof(double) * a.m * a.m, (most - (int)sizeof(Shared<RR>)) / 256 * 256);
    GS2_TRY_HIP(hipFuncSetAttribute((const void *)k_resident<VT, AT, KL, RR>, hipFuncAttributeMaxDynamicSharedMemorySize, a.lds));
    k_resident<VT, AT, KL, RR><<<(unsigned)a.G, threads_of(RR), (size_t)a.lds, s>>>(a);
    GS2_TRY_HIP(hipGetLastError());
    return GS2_OK;
}

template <typename VT, typename AT, int KL>
int launch_lanes(const ResArgs &a, hipStream_t s)
{
    switch (res_rows(a.n)) {
    case 256: return launch_rows<VT, AT, KL, 256>(a, s);
    case 512: return launch_rows<VT, AT, KL, 512>(a, s);
    default:
        if constexpr (KL < 2) return launch_rows<VT, AT, KL, 1024>(a, s);
        return GS2_ERR_ARG; // res_lanes
    }
}

template <typename VT, typename AT>
int launch(int sum_lanes, const ResArgs &a, hipStream_t s)
{
    return sum_lanes == 1   ? launch_lanes<VT, AT, 0>(a, s)
           : sum_lanes == 2 ? launch_lanes<VT, AT, 1>(a, s)
                            : launch_lanes<VT, AT, 2>(a, s);
}

} // namespace

int resident_launch(int precision, int sum_lanes, const ResArgs &a, hipStream_t s)
{
    return precision == GS2_FP64   ? launch<double, double>(sum_lanes, a, s)
           : precision == GS2_FP32 ? launch<float, float>(sum_lanes, a, s)
                                   : launch<_Float16, float>(sum_lanes, a, s);
}

} // namespace gs2
