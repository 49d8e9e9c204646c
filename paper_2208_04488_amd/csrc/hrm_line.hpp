// hrm_line.hpp -- launches of the line kernels (hrm_line.hip).
#pragma once

#include "hrm.h"
#include "hrm_device.hpp"

namespace hrm {

// the first-order schemes in double (the float one runs in the general kernel)
inline bool line_first_order(int flags, int precision)
{
    return (flags & F_FOUR_EQ) || ((flags & F_FIRST_ORDER) && precision == HRM_FP64);
}

// Cells of the longest line that one workgroup advances, a face per thread.
// Beyond, a launch per step on several CUs with one wave of faces on a SIMD is
// faster than two on each of one CU's (us a step, this against those: high order,
// two species, 447 cells 21.3 / 25.0, 480 26.7 / 24.5; three species, 320 cells 30.5
// / 35.1, 447 38.1 / 35.7; four equations, 511 cells 10.0 / 11.9, 600 13.5 / 12.0).
inline int line_cells(int N, int flags, int precision)
{
    return line_first_order(flags, precision) ? 511 : (N == 2 ? 447 : 383);
}

struct LineArgs {
    double* W;     // state (M x n), in/out
    double* slot;  // dt, lambda_0..2, t
    unsigned long long* cnt;
    int n, nsteps;
    int bclo, bchi;
    const double* blo;  // Dirichlet ghost state of the low / high end (M), or null
    const double* bhi;
    double idx;
    DtArgs dt;
    EosDev e;
    ParDev P;
};

// Steps of one launch.  A long run is many launches of a few milliseconds (256
// steps of 400 cells 5.5 ms), so that other work of the device comes between them
// and the state is in memory at each end; the state and the time carry over to
// the bit, and a launch costs 0.1 % of its steps.
constexpr int LINE_STEPS = 256;

// N = 2 or 3, 1 <= A.n <= line_cells(N, ...)
void line_launch(int N, int precision, const LineArgs& A, hipStream_t s);

// the steps of a longer line, a launch each, in tiles of LINE_BS threads
constexpr int LINE_BS = 256;

// Lines advanced without the sweeps: up to where the tiles fill the chip and their
// halos cost more than the launches (us a step, a launch each against three sweeps:
// 5000 cells 23.6 / 31.7, 120000 32.4 / 42.0, 300000 54.7 / 62.9; three species,
// 600000 139.5 / 136.0).  The learned weights are left to the sweeps.
inline bool line_fits(int n, int flags, int precision, int weights)
{
    return n <= 1200 * LINE_BS && (line_first_order(flags, precision) || weights == HRM_WEIGHTS_IS);
}

// doubles of `part` (wavespeeds of two steps and the time) for n cells
inline long long line_part(long long n) { return 2 * (n / (LINE_BS / 2) + 2) + 2; }

struct LineStepArgs {
    LineArgs a;  // first: line_nodes and line_update find its members there
    const double* src;
    double* dst;
    const double* pin;  // wavespeeds of src, by tile
    double* pout;       // those of dst (null after the last step)
    const double* tin;
    double* tout;
    int own, npart;
};

// N = 2 or 3, line_fits(A.n, ...); other: as many doubles as the state
void line_steps(int N, int precision, const LineArgs& A, double* other, double* part, hipStream_t s);

}  // namespace hrm
