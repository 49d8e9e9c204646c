// hrm_line.hpp -- launch of the one-workgroup advance of a short line
// (hrm_line.hip).
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
// Up to 511 it beats a launch per sweep on several CUs at every scheme.  From
// 512 on the four SIMDs of one CU have four waves of faces each and are
// slower than several CUs for the high-order scheme (two species, a step: 29
// against 35 us at 400 cells, 38 against 35 at 700), but not for the
// first-order schemes, whose faces are a tenth of the work (four equations: 16
// against 25 us at 1023).
inline int line_cells(int flags, int precision, int weights)
{
    if (line_first_order(flags, precision)) return 1023;
    return weights == HRM_WEIGHTS_IS ? 511 : 0;
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

// N = 2 or 3, 1 <= A.n <= line_cells()
void line_launch(int N, int precision, const LineArgs& A, hipStream_t s);

}  // namespace hrm
