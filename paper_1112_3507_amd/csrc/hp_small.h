// hp_small.h -- interface of the one-launch V-cycles and CG solves of hp_small.hip.
#pragma once

#include "hp_internal.h"

namespace hp {

constexpr int kSmallThreads = 512;              // a workgroup (1024 leave 64 registers a lane: 300 spills)
constexpr int kSmallLevels = 16;                // most levels one launch takes
constexpr int kSmallItems = 4 * kSmallThreads;  // most x pairs of its first level: four of each colour per thread
constexpr int kSmallLds = 159 * 1024;           // LDS bytes for its vectors
constexpr int kBarrierPolls = 1 << 22;          // seconds: only a lost member could make a barrier last that long

// Counters of a launch, all zero before it (and again after it); one launch at a time.
struct SmallState {
    unsigned joined, size, left, done, pad0[28];
    unsigned arrived, pad1[31];  // on a cache line of its own: every barrier polls it
};

struct SmallLevel {
    Geo<double> g;
    int coarsened[3], periodic[3];  // towards the next level, per axis (as in Transfer)
    int n, hx, items;               // cells; ceil(nx / 2); cells of one colour, rows of hx
    int lds;                        // below the first level: where its r, z, t start in LDS (values behind the first's)
    float inv_nx, inv_hx, inv_ny;   // reciprocals of the row lengths and row counts
    float c32[3];                   // the FP32 face factors
    const double *rho, *m;
    double* dinv;
    float* dinv32;
    double* w;  // weights of the high faces, three arrays of n (none on the coarsest level)
};

// The levels that these launches run on, in device memory (the last one is the coarsest): a launch's
// own arguments lie in host memory, where every look at them costs.
struct SmallTable {
    SmallLevel lv[kSmallLevels];
    const double* ainv;
    int levels, nc;
};
static_assert(sizeof(SmallTable) <= 4000, "a kernel's arguments");

// How a solve ended. SMALL_INPUT: b or x is not finite; SMALL_LOST: a barrier ran out of polls.
enum { SMALL_MORE = 0, SMALL_CONVERGED, SMALL_BUDGET, SMALL_BREAKDOWN, SMALL_NAN, SMALL_INPUT, SMALL_LOST };

// What a solve leaves (host memory the device writes): the squared true residual norm and ||b||^2, the
// iterations, the rounds after the first, the code.
struct SmallResult {
    double rr, bb;
    int iterations, rounds, code, pad;
};

// Solve of A x = b by CG from x, in natural order, to the true residual tol ||b|| or `budget` iterations;
// every round starts from the true residual.
struct SmallCG {
    double* x;
    const double* b;
    SmallResult* result;
    double tol;
    int budget;
};

struct SmallArgs {
    const SmallTable* table;
    int nu_pre, nu_post;
    const double* r;   // the first level's right-hand side
    double* z;         // where a V-cycle's result goes
    double* exchange;  // 2 nc values between the owner and its helpers
    SmallState* state;
    double* scal;      // if a V-cycle's barrier ran out of polls, S_FLAG is FLAG_LOST, and z NaN
    int polls;
    SmallCG cg;
};

struct SmallShape {
    int groups = 0;      // workgroups: the owner and the helpers of its coarsest solve
    int per_thread = 0;  // items of a colour per thread on the first level
    int lds_cycle = 0;   // LDS vectors of a V-cycle, in values
    int lds_cg = 0;      // and of a whole solve (0: too large for one launch)
};

// Before the first launch of this shape on the device.
hipError_t prepare_small(const SmallShape& sh);

// One V-cycle from r to z, or (whole_cg) the solve a.cg.
void launch_small(const SmallArgs& a, bool whole_cg, const SmallShape& sh, hipStream_t s);

// Writes the table to the device, and computes the Jacobi diagonals (FP64 and FP32) of its levels and the
// face weights of all but the coarsest, each in its level's storage order.
void launch_small_setup(const SmallTable& a, int face_rule, SmallTable* table, hipStream_t s);

}  // namespace hp
