// hrm_line.hip -- SSP-RK3 steps of one line (1D grid) with all stages in one
// launch (gfx950): the smallest grids, whose steps are launch and latency bound.
//
// k_line: many steps of a short line in one workgroup.  A thread owns a cell, whose
// state stays in registers from the first step to the last, and the face on its
// low side.  The node records of a stage and the
// face fluxes are exchanged through LDS, the time step by a reduction over the
// workgroup, so a step needs neither memory nor another launch: two species,
// high order, a step of 256 / 400 cells 21.6 / 20.7 us against 35 as four launches
// (a reduction and three sweeps); four equations, 400 cells 9.9 against 25 us.
// k_line_step: a longer line in tiles, a launch per step.  The arithmetic is
// k_sweep's, in the order that the shared functions write out (hrm_device.hpp),
// and so are the bits.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>

#include "hrm.h"
#include "hrm_face.hpp"
#include "hrm_line.hpp"

namespace hrm {

// Node records of a line of n cells, one a thread, and of the three ghost nodes
// at both ends: m is the thread's |u| + c, mg that of a Dirichlet state.  LOW as
// face_flux takes it; the arguments start with a LineArgs.
template <int N, int FS, int LOW>
__device__ __forceinline__ void line_nodes(double* lds, int ts, int n, int bclo, int bchi, const double* blo,
                                           const double* bhi, bool four, const double* w, double& m, double& mg)
{
    constexpr int D = 1, M = 2 * N + D;
    using F = NodeFields<N, D>;
    const EosDev e = kload<EosDev>(kernel_args() + offsetof(LineArgs, e));
    auto store_node = [&](const double* W, const St<N, D>& s, int l) {
#pragma unroll
        for (int c = 0; c < M; ++c) lds[c * FS + l] = W[c];
        lds[F::U * FS + l] = s.u[0];
        lds[F::P * FS + l] = s.p;
        lds[F::RHO * FS + l] = s.rho;
        lds[F::C * FS + l] = s.c;
    };
    auto node_state = [&](const double* W, St<N, D>& s) {
        state_from_W<N, D>(e, W, s);
        if constexpr (LOW == 2)
            if (four) hrm4_pc<N, D>(e, s, s.p, s.c);
    };
    m = mg = 0.0;
    if (ts < n) {
        St<N, D> s;
        node_state(w, s);
        store_node(w, s, ts + 3);
        m = fabs(s.u[0]) + s.c;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int g = q < 3 ? q - 3 : n + q - 3;
            if ((q < 3 ? bclo : bchi) != BC_DIRICHLET && map_bc(g, n, bclo, bchi) == ts) store_node(w, s, g + 3);
        }
    }
    if (bclo == BC_DIRICHLET || bchi == BC_DIRICHLET) {
        // ghost node ts of the six; its state counts for the time step
        const double* src =
            ts < 3 ? (bclo == BC_DIRICHLET ? blo : nullptr) : (ts < 6 && bchi == BC_DIRICHLET ? bhi : nullptr);
        if (src) {
            double W[M];
#pragma unroll
            for (int c = 0; c < M; ++c) W[c] = src[c];
            St<N, D> s;
            node_state(W, s);
            store_node(W, s, ts < 3 ? ts : n + ts);
            mg = fabs(s.u[0]) + s.c;
        }
    }
}

// Fluxes of the faces 0 .. n and the stage update of the cells 0 .. n-1, with
// the relaxation.  The workgroup's threads come here together.
template <int N, int FS, typename R, int LOW>
__device__ __forceinline__ void line_update(double* lds, int ts, int n, int stage, double dt, double lam, double idx,
                                            bool count_face, bool count_cell, const double* Wn, double* w,
                                            unsigned long long* counters)
{
    constexpr int D = 1, M = 2 * N + D, IA = N + D + 1;
    constexpr int NA = N > 1 ? N - 1 : 1;
    // waves whose faces all lie beyond face n only take part in the barriers
    const bool live = __builtin_amdgcn_readfirstlane(ts & ~63) <= n;
    double G[M], Gp[NA];
    unsigned cnt = 0;
    if (live) {
        unsigned lc = 0;
        const KArg ka = kernel_args();
        // lanes beyond face n repeat it: whatever LDS holds there would
        // send the whole wave through the limiters' rare paths
        face_flux<N, D, 0, 1, FS, R, 0, LOW>(lds + min(ts, n), ka + offsetof(LineArgs, e), ka + offsetof(LineArgs, P),
                                             lam, G, Gp, lc);
        if (count_face) cnt = lc;
    }
    __syncthreads();
    if (live) {
#pragma unroll
        for (int c = 0; c < M; ++c) lds[c * FS + ts] = G[c];
#pragma unroll
        for (int k = 0; k < N - 1; ++k) lds[(M + k) * FS + ts] = Gp[k];
    }
    __syncthreads();
    if (ts < n) {
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
                w[c] = stage_value(ca, cb, Wn[c], w[c], dt, flux_difference(lds[c * FS + ts + 1], gm, idx));
            }
            if (!relax_cell<N, D>(kload<EosDev>(kernel_args() + offsetof(LineArgs, e)), w) && count_cell)
                cnt += cnt_one(C_RELAX_BAD);
        }
    }
    flush_counters(cnt, counters);
    __syncthreads();
}

template <int N, int BS, typename R, int LOW>
__global__ void __launch_bounds__(BS) k_line(const LineArgs A)
{
    constexpr int D = 1, M = 2 * N + D;
    constexpr int FS = BS + 5, NW = BS / 64;
    __shared__ double lds[NodeFields<N, D>::COUNT * FS];
    __shared__ double sh[NW];
    const int ts = threadIdx.x, n = A.n;
    const bool cell = ts < n;
    [[maybe_unused]] const bool four = (A.P.flags & F_FOUR_EQ) != 0;

    double w[M], Wn[M];
    if (cell)
#pragma unroll
        for (int c = 0; c < M; ++c) w[c] = A.W[(long long)c * n + ts];

    double slot[5] = {0.0, 0.0, 0.0, 0.0, A.slot[4]};
    for (int step = 0; step < A.nsteps; ++step) {
#pragma unroll 1
        for (int stage = 0; stage < 3; ++stage) {
            double m, mg;
            line_nodes<N, FS, LOW>(lds, ts, n, A.bclo, A.bchi, A.blo, A.bhi, four, w, m, mg);
            if (stage == 0) {
                // Sec. 4.1.2: every wave leaves its maximum, every thread
                // takes the maximum of those and forms the same time step
                m = nmax(m, mg);
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
            line_update<N, FS, R, LOW>(lds, ts, n, stage, slot[0], slot[1], A.idx, ts <= n, true, Wn, w, A.cnt);
        }
    }
    if (cell)
#pragma unroll
        for (int c = 0; c < M; ++c) A.W[(long long)c * n + ts] = w[c];
    if (ts == 0)
#pragma unroll
        for (int i = 0; i < 5; ++i) A.slot[i] = slot[i];
}

// One step of a longer line, all three stages in one launch: a workgroup takes
// `own` cells and the cells on both sides that its own ones depend on over three
// stages (nine, or three at first order), and advances them all.  The cells at
// an inner end of the tile see a copy of the last one instead of their
// neighbours and are wrong by as much as the halo is wide.  Bound by the latency
// of three stages, one wave of faces on a SIMD; a launch a sweep took a launch
// and a pass through memory more per stage.  us a step, three sweeps -> this: four
// equations, 5000 cells 22.2 -> 12.0; high order, 5000 cells 31.7 -> 23.6, three
// species 43.5 -> 33.8, 120000 cells 42.0 -> 32.4.
template <int N, int BS, typename R, int LOW>
__global__ void __launch_bounds__(BS) k_line_step(const LineStepArgs A)
{
    constexpr int D = 1, M = 2 * N + D, H = LOW == 2 ? 3 : 9;
    constexpr int FS = BS + 5, NW = BS / 64;
    __shared__ double lds[NodeFields<N, D>::COUNT * FS];
    __shared__ double sh[NW];
    const int ts = threadIdx.x, n = A.a.n;
    const bool periodic = A.a.bclo == BC_PERIODIC;
    const int c0 = blockIdx.x * A.own, c1 = min(c0 + A.own, n);
    // cells e0 .. e1-1; indices beyond the ends of a periodic line wrap
    const int e0 = periodic ? c0 - H : max(c0 - H, 0), e1 = periodic ? c1 + H : min(c1 + H, n);
    const int ne = e1 - e0, g = e0 + ts;
    const int bclo = !periodic && e0 == 0 ? A.a.bclo : 0, bchi = !periodic && e1 == n ? A.a.bchi : 0;
    const bool four = (A.a.P.flags & F_FOUR_EQ) != 0, owned = g >= c0 && g < c1;

    double w[M], Wn[M];
    if (ts < ne) {
        const int i = map_bc(g, n, 1, 1);
#pragma unroll
        for (int c = 0; c < M; ++c) Wn[c] = w[c] = A.src[(long long)c * n + i];
    }
    double m = 0.0, mg, slot[5] = {0.0, 0.0, 0.0, 0.0, *A.tin};
    for (int i = ts; i < A.npart; i += BS) m = nmax(m, A.pin[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = nmax(m, __shfl_xor(m, off, 64));
    if ((ts & 63) == 0) sh[ts >> 6] = m;
#pragma unroll 1
    for (int stage = 0; stage < 3; ++stage) {
        line_nodes<N, FS, LOW>(lds, ts, ne, bclo, bchi, A.a.blo, A.a.bhi, four, w, m, mg);
        __syncthreads();
        if (stage == 0) {
            double mx = sh[0];
#pragma unroll
            for (int i = 1; i < NW; ++i) mx = nmax(mx, sh[i]);
            dt_from_max(&mx, A.a.dt, slot);
        }
        line_update<N, FS, R, LOW>(lds, ts, ne, stage, slot[0], slot[1], A.a.idx, owned || (g == n && c1 == n), owned,
                                   Wn, w, A.a.cnt);
    }
    if (owned) {
#pragma unroll
        for (int c = 0; c < M; ++c) A.dst[(long long)c * n + g] = w[c];
    }
    // the wavespeeds of the new state, for the next step
    if (A.pout) {
        line_nodes<N, FS, LOW>(lds, ts, ne, bclo, bchi, A.a.blo, A.a.bhi, four, w, m, mg);
        m = nmax(owned ? m : 0.0, mg);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = nmax(m, __shfl_xor(m, off, 64));
        if ((ts & 63) == 0) sh[ts >> 6] = m;
        __syncthreads();
        if (ts == 0) {
#pragma unroll
            for (int i = 1; i < NW; ++i) m = nmax(m, sh[i]);
            A.pout[blockIdx.x] = m;
        }
    }
    if (ts == 0 && blockIdx.x == 0) {
        *A.tout = slot[4];
#pragma unroll
        for (int i = 0; i < 5; ++i) A.a.slot[i] = slot[i];
    }
}

// before the first of those steps: the wavespeeds of W (and of a Dirichlet
// state, in the end tiles), the time, and for an odd number of steps, which go
// to and fro between two buffers, a copy of W
template <int N>
__global__ void __launch_bounds__(256) k_line_start(const LineStepArgs A)
{
    constexpr int D = 1, M = 2 * N + D;
    __shared__ double sh[4];
    const int ts = threadIdx.x, n = A.a.n, c0 = blockIdx.x * A.own, c1 = min(c0 + A.own, n);
    const bool four = (A.a.P.flags & F_FOUR_EQ) != 0;
    const EosDev& e = A.a.e;
    double m = 0.0;
    auto take = [&](const double* W) {
        St<N, D> s;
        state_from_W<N, D>(e, W, s);
        double p, c = s.c;
        if (four) hrm4_pc<N, D>(e, s, p, c);
        m = nmax(m, fabs(s.u[0]) + c);
    };
    for (int i = c0 + ts; i < c1; i += 256) {
        double w[M];
#pragma unroll
        for (int c = 0; c < M; ++c) w[c] = A.src[(long long)c * n + i];
        take(w);
        if (A.dst)
#pragma unroll
            for (int c = 0; c < M; ++c) A.dst[(long long)c * n + i] = w[c];
    }
    const double* b = ts == 0 && c0 == 0 && A.a.bclo == BC_DIRICHLET ? A.a.blo
                      : ts == 1 && c1 == n && A.a.bchi == BC_DIRICHLET ? A.a.bhi : nullptr;
    if (b) take(b);
    block_max<1>(&m, sh);
    if (ts == 0) {
        A.pout[blockIdx.x] = m;
        if (blockIdx.x == 0) *A.tout = A.a.slot[4];
    }
}

namespace {

template <int N, typename R, int LOW>
void launch(const LineArgs& A, hipStream_t s)
{
    if (A.n < 256)
        hipLaunchKernelGGL((k_line<N, 256, R, LOW>), dim3(1), dim3(256), 0, s, A);
    else
        hipLaunchKernelGGL((k_line<N, 512, R, LOW>), dim3(1), dim3(512), 0, s, A);
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

template <int N, typename R, int LOW>
void launch_step(const LineStepArgs& A, int tiles, hipStream_t s)
{
    hipLaunchKernelGGL((k_line_step<N, LINE_BS, R, LOW>), dim3(tiles), dim3(LINE_BS), 0, s, A);
}

template <int N>
void launch_steps(int precision, const LineArgs& L, double* other, double* part, hipStream_t s)
{
    const bool low = line_first_order(L.P.flags, precision);
    const int most = LINE_BS - 1 - 2 * (low ? 3 : 9);
    const int tiles = (L.n + most - 1) / most;
    LineStepArgs A;
    memset(&A, 0, sizeof(A));
    A.a = L;
    A.own = (L.n + tiles - 1) / tiles;
    A.npart = (L.n + A.own - 1) / A.own;
    double* const buf[2] = {L.nsteps % 2 ? other : L.W, L.nsteps % 2 ? L.W : other};
    double *const p[2] = {part, part + A.npart}, *const t = part + 2 * A.npart;
    A.src = L.W;
    A.dst = L.nsteps % 2 ? other : nullptr;
    A.pout = p[0];
    A.tout = t;
    hipLaunchKernelGGL((k_line_start<N>), dim3(A.npart), dim3(256), 0, s, A);
    for (int k = 0; k < L.nsteps; ++k) {
        A.src = buf[k % 2];
        A.dst = buf[(k + 1) % 2];
        A.pin = p[k % 2];
        A.pout = k + 1 < L.nsteps ? p[(k + 1) % 2] : nullptr;
        A.tin = t + k % 2;
        A.tout = t + (k + 1) % 2;
        if (low)
            launch_step<N, double, 2>(A, A.npart, s);
        else if (precision == HRM_FP32)
            launch_step<N, float, 1>(A, A.npart, s);
        else
            launch_step<N, double, 0>(A, A.npart, s);
    }
}

}  // namespace

void line_launch(int N, int precision, const LineArgs& A, hipStream_t s)
{
    LineArgs part = A;
    for (int done = 0; done < A.nsteps; done += part.nsteps) {
        part.nsteps = A.nsteps - done < LINE_STEPS ? A.nsteps - done : LINE_STEPS;
        if (N == 2)
            launch_n<2>(precision, part, s);
        else
            launch_n<3>(precision, part, s);
    }
}

void line_steps(int N, int precision, const LineArgs& A, double* other, double* part, hipStream_t s)
{
    if (N == 2)
        launch_steps<2>(precision, A, other, part, s);
    else
        launch_steps<3>(precision, A, other, part, s);
}

}  // namespace hrm
