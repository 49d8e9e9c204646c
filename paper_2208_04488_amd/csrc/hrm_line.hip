// hrm_line.hip -- SSP-RK3 steps of one short line (1D grid) in one workgroup
// (gfx950): the smallest grids, whose steps are launch and latency bound.
//
// A thread owns a cell, whose state stays in registers from the first step to
// the last, and the face on its low side.  The node records of a stage and the
// face fluxes are exchanged through LDS, the time step by a reduction over the
// workgroup, so a step needs neither memory nor another launch: two species,
// high order, a step of 100 / 400 / 511 cells 24 / 28 / 25 us against 35 as four
// launches (a reduction and three sweeps); four equations, 400 / 1023 cells
// 10 / 16 against 25 us.  The arithmetic is k_sweep's, in the same
// order, and so are the bits.
#include <hip/hip_runtime.h>

#include <cstddef>

#include "hrm.h"
#include "hrm_face.hpp"
#include "hrm_line.hpp"

namespace hrm {

// LOW as face_flux takes it
template <int N, int BS, typename R, int LOW>
__global__ void __launch_bounds__(BS) k_line(const LineArgs A)
{
    constexpr int D = 1;
    using F = NodeFields<N, D>;
    constexpr int M = 2 * N + D, IA = N + D + 1;
    constexpr int NA = N > 1 ? N - 1 : 1;
    constexpr int FS = BS + 5, NW = BS / 64;
    __shared__ double lds[F::COUNT * FS];
    __shared__ double sh[NW];
    const int ts = threadIdx.x, n = A.n;
    const bool cell = ts < n;
    [[maybe_unused]] const bool four = (A.P.flags & F_FOUR_EQ) != 0;
    // waves whose faces all lie beyond face n only take part in the barriers
    const bool live = __builtin_amdgcn_readfirstlane(ts & ~63) <= n;

    double w[M], Wn[M];
    if (cell)
#pragma unroll
        for (int c = 0; c < M; ++c) w[c] = A.W[(long long)c * n + ts];

    auto store_node = [&](const EosDev& e, const double* W, const St<N, D>& s, int l) {
#pragma unroll
        for (int c = 0; c < M; ++c) lds[c * FS + l] = W[c];
        lds[F::U * FS + l] = s.u[0];
        lds[F::P * FS + l] = s.p;
        lds[F::RHO * FS + l] = s.rho;
        lds[F::C * FS + l] = s.c;
    };
    auto node_state = [&](const EosDev& e, const double* W, St<N, D>& s) {
        state_from_W<N, D>(e, W, s);
        if constexpr (LOW == 2)
            if (four) hrm4_pc<N, D>(e, s, s.p, s.c);
    };

    double slot[5] = {0.0, 0.0, 0.0, 0.0, A.slot[4]};
    for (int step = 0; step < A.nsteps; ++step) {
#pragma unroll 1
        for (int stage = 0; stage < 3; ++stage) {
            // node records of the line and of the ghost nodes at both ends
            double m = 0.0;
            {
                const EosDev e = kload<EosDev>(kernel_args() + offsetof(LineArgs, e));
                if (cell) {
                    St<N, D> s;
                    node_state(e, w, s);
                    store_node(e, w, s, ts + 3);
                    m = fabs(s.u[0]) + s.c;
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        const int g = q < 3 ? q - 3 : n + q - 3;
                        if ((q < 3 ? A.bclo : A.bchi) != BC_DIRICHLET && map_bc(g, n, A.bclo, A.bchi) == ts)
                            store_node(e, w, s, g + 3);
                    }
                }
                if (A.bclo == BC_DIRICHLET || A.bchi == BC_DIRICHLET) {
                    // ghost node ts of the six; its state counts for the time step
                    const double* src = ts < 3 ? (A.bclo == BC_DIRICHLET ? A.blo : nullptr)
                                               : (ts < 6 && A.bchi == BC_DIRICHLET ? A.bhi : nullptr);
                    if (src) {
                        double W[M];
#pragma unroll
                        for (int c = 0; c < M; ++c) W[c] = src[c];
                        St<N, D> s;
                        node_state(e, W, s);
                        store_node(e, W, s, ts < 3 ? ts : n + ts);
                        m = nmax(m, fabs(s.u[0]) + s.c);
                    }
                }
            }
            if (stage == 0) {
                // Sec. 4.1.2: every wave leaves its maximum, every thread
                // takes the maximum of those and forms the same time step
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) m = nmax(m, __shfl_xor(m, off, 64));
                if ((ts & 63) == 0) sh[ts >> 6] = m;
#pragma unroll
                for (int c = 0; c < M; ++c) Wn[c] = w[c];
            }
            __syncthreads();
            if (stage == 0) {
                double mx = sh[0];
#pragma unroll
                for (int i = 1; i < NW; ++i) mx = nmax(mx, sh[i]);
                dt_from_max(&mx, A.dt, slot);
            }
            const double dt = slot[0];
            double G[M], Gp[NA];
            unsigned cnt = 0;
            if (live) {
                unsigned lc = 0;
                const KArg ka = kernel_args();
                // lanes beyond face n repeat it: whatever LDS holds there would
                // send the whole wave through the limiters' rare paths
                face_flux<N, D, 0, 1, FS, R, 0, LOW>(lds + min(ts, n), ka + offsetof(LineArgs, e), ka + offsetof(LineArgs, P), slot[1],
                                             G, Gp, lc);
                if (ts <= n) cnt = lc;
            }
            __syncthreads();
            if (live) {
#pragma unroll
                for (int c = 0; c < M; ++c) lds[c * FS + ts] = G[c];
#pragma unroll
                for (int k = 0; k < N - 1; ++k) lds[(M + k) * FS + ts] = Gp[k];
            }
            __syncthreads();
            if (cell) {
                // Shu-Osher coefficients (a, b) of the three stages
                const double ca = stage == 0 ? 0.0 : (stage == 1 ? 3.0 / 4.0 : 1.0 / 3.0);
                const double cb = stage == 0 ? 1.0 : (stage == 1 ? 1.0 / 4.0 : 2.0 / 3.0);
                if (__builtin_expect(dt == 0.0, 0)) {
                    // held at the end time: W^n as it is
#pragma unroll
                    for (int c = 0; c < M; ++c) w[c] = Wn[c];
                } else {
#pragma unroll
                    for (int c = 0; c < M; ++c) {
                        const double gm = c >= IA ? lds[(M + c - IA) * FS + ts] : lds[c * FS + ts];
                        const double L = -(lds[c * FS + ts + 1] - gm) * A.idx;
                        w[c] = ca * Wn[c] + cb * (w[c] + dt * L);
                    }
                    if (!relax_cell<N, D>(kload<EosDev>(kernel_args() + offsetof(LineArgs, e)), w))
                        cnt += cnt_one(C_RELAX_BAD);
                }
            }
            flush_counters(cnt, A.cnt);
            __syncthreads();
        }
    }
    if (cell)
#pragma unroll
        for (int c = 0; c < M; ++c) A.W[(long long)c * n + ts] = w[c];
    if (ts == 0)
#pragma unroll
        for (int i = 0; i < 5; ++i) A.slot[i] = slot[i];
}

namespace {

template <int N, typename R, int LOW>
void launch(const LineArgs& A, hipStream_t s)
{
    if (A.n < 256)
        hipLaunchKernelGGL((k_line<N, 256, R, LOW>), dim3(1), dim3(256), 0, s, A);
    else if (A.n < 512)
        hipLaunchKernelGGL((k_line<N, 512, R, LOW>), dim3(1), dim3(512), 0, s, A);
    else if constexpr (LOW == 2)
        hipLaunchKernelGGL((k_line<N, 1024, R, LOW>), dim3(1), dim3(1024), 0, s, A);
}

template <int N>
void launch_n(int precision, const LineArgs& A, hipStream_t s)
{
    if (line_first_order(A.P.flags, precision))
        launch<N, double, 2>(A, s);
    else if (precision == HRM_FP32)
        launch<N, float, 1>(A, s);
    else
        launch<N, double, 0>(A, s);
}

}  // namespace

void line_launch(int N, int precision, const LineArgs& A, hipStream_t s)
{
    if (N == 2)
        launch_n<2>(precision, A, s);
    else
        launch_n<3>(precision, A, s);
}

}  // namespace hrm
