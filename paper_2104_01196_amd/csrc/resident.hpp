// The one-launch GMRES solve of small systems (resident.hip).
#pragma once

#include "gs2_internal.hpp"

namespace gs2 {

constexpr int RES_MAX_GROUPS = 64;  // workgroups of one solve: a partial sum per lane
constexpr int RES_MAX_ROWS = 1024;  // rows per workgroup, at most
constexpr int RES_MAX_EX = 32;      // most vectors exchanged within a preconditioner apply
constexpr int64_t RES_MAX_N = (int64_t)RES_MAX_GROUPS * RES_MAX_ROWS;
constexpr int RES_MAX_M = 64;       // longest restart (its Hessenberg matrix sits in LDS)
constexpr unsigned RES_WAIT_POLLS = 1u << 21; // trips to memory before a wait ends, half a microsecond or more each
constexpr int RES_GIVEN_UP = 1000;  // ResInfo::status of a solve whose wait ran out

// Rows per workgroup of a small system, here and where it is solved launch by
// launch: the fewest that RES_MAX_GROUPS workgroups hold.
inline int res_rows(int64_t n)
{
    int r = 256;
    while (r < RES_MAX_ROWS && n > (int64_t)RES_MAX_GROUPS * r) r *= 2;
    return r;
}

// Most lanes per row whose sums it can repeat: as the registers of a row's thread
// allow.
inline int res_lanes(int64_t n) { return res_rows(n) < RES_MAX_ROWS ? 4 : 2; }

// A sliced-ELL matrix, 2^lk lanes per row.
struct ResSell {
    const int64_t *sp;
    const int32_t *col;
    const void *val;
    int lk;
};

struct ResInfo {
    int iterations, restarts, status, converged;
    double relres;
};

struct ResArgs {
    int n, G, m, maxit, stag, kind;
    int sweeps, inner, variant, compact;
    int lds; // bytes of dynamic LDS (resident_launch)
    double rtol, omega, gamma;
    ResSell L, U, A;
    const double *sl, *sr, *b;
    double *x;
    double *V, *Z;              // own rows only: plain accesses
    // exchanged between workgroups, agent scope only: x; z, two turns; S_l u and
    // the preconditioner's ne vectors, two turns; partial sums (res_parts)
    double *xe, *ze;
    void *ex;
    int ne;
    double *part;
    unsigned *bar; // arrivals, abort, departures: zero between solves
    unsigned looks; // before a wait ends
    ResInfo *info;
};

// partial sums per workgroup: one of a norm between barriers, and three turns
// of a step's norm and its first pass's sums
constexpr int res_parts(int m) { return 1 + 3 * (1 + 2 * m + 3); }

// sum_lanes: lanes per row whose sums the launched passes add (1 for the
// layouts that add a row's entries one after the other)
int resident_launch(int precision, int sum_lanes, const ResArgs &a, hipStream_t s);

} // namespace gs2
