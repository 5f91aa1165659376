// The one-launch GMRES solve of small systems (resident.hip).
#pragma once

#include "gs2_internal.hpp"

namespace gs2 {

constexpr int RES_MAX_GROUPS = 64;  // workgroups of one solve: a partial sum per lane
constexpr int RES_ROWS = 1024;      // rows per workgroup
constexpr int RES_MAX_LANES = 4;    // lanes per row whose sums it can repeat
constexpr int64_t RES_MAX_N = (int64_t)RES_MAX_GROUPS * RES_ROWS;
constexpr int RES_MAX_M = 64;       // longest restart (its Hessenberg matrix sits in LDS)
constexpr int RES_GIVEN_UP = 1000;  // ResInfo::status of a solve whose wait ran out

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
    void *se;                   // exchanged, as xh .. gb: agent scope only
    double *ze, *xe, *part;
    void *xh, *xh2, *rh, *ga, *gb;
    unsigned *bar; // arrivals, abort, departures: zero between solves
    ResInfo *info;
};

// sum_lanes: lanes per row whose sums the launched passes add (1 for the
// layouts that add a row's entries one after the other)
int resident_launch(int precision, int sum_lanes, const ResArgs &a, hipStream_t s);

} // namespace gs2
