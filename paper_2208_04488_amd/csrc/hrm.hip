// hrm.hip -- gfx950 kernels and the C-ABI of the PP-WCNS-IS stage and the
// thermal relaxation (arXiv:2208.04488).  Declarations and semantics of the
// exported calls are in include/hrm.h.
//
// Kernels
//   k_sweep<N,D,DIR>  one direction of the spatial operator.  A block stages
//                     the primitive data of a tile of nodes (with the 3-node
//                     halo on both sides, boundary conditions applied at load)
//                     in LDS, computes one face per thread, writes the face
//                     pairs back to LDS and forms the flux difference of each
//                     cell.  The last direction also applies the Shu-Osher
//                     stage update and, optionally, the relaxation; in the
//                     last stage of a step it also folds the block maxima
//                     of |u_d| + c of the new state into the partial slots
//                     of the next step's time step.
//   k_plane           a stage of a small 2D grid, both directions of a tile.
//   k_relax           point-wise relaxation.
//   k_wavespeed       per-block max of |u_d| + c (the first step of a run,
//                     hrm_max_wavespeed), then k_reduce_max / k_reduce_dt
//                     (which clears the slots the sweep folds into).
//   k_dt              the time step and lambda_d on the device.
// Lines take other kernels (hrm_line.hip): short ones all steps in one workgroup,
// longer ones a launch per step (line_cells, line_fits).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <new>

#include "hrm.h"
#include "hrm_face.hpp"
#include "hrm_line.hpp"

namespace hrm {

struct SweepArgs {
    const double* Ws;
    const double* Wn;
    double* Wout;
    double* rhs;
    const double* slot;
    unsigned long long* cnt;
    long long ncell;
    int n[3];
    int bclo, bchi;
    const double* blo;  // Dirichlet ghost states of the low / high face (M x face cells), or null
    const double* bhi;
    double* wpart;  // mode 2, non-null: maxima of |u_d| + c of the stage output, block b into slot b % nslot
    unsigned nslot; // a power of two, at most the number of blocks
    unsigned rnp;   // packed lines: floor(2^32 / (n[0] + 1)), or 0 from 2^32 faces on
    int mode;  // 0: rhs = L_d, 1: rhs += L_d, 2: stage update with rhs + L_d
    int relax;
    int hold;  // mode 2 within a full RK3 step: a step of dt = 0 (the end time reached) leaves W^n as it is
    double a, b;
    double idx;
    // lines (D = 1), a step's first two sweeps (phase 1, 2; 0 elsewhere)
    int phase, npart;
    double* part;   // wavespeed partials of W^n (npart, the first nslot cleared for the step's last sweep)
    double* tnext;  // the time after the step, from phase 1 to phase 2
    double* slotw;  // `slot`, to write
    DtArgs dt;
    EosDev e;
    ParDev P;
};

constexpr int MODE_WRITE = 0, MODE_ADD = 1, MODE_FINAL = 2;

// one DPP move of a 64-bit value (both halves with the same control); rows
// outside ROWS keep their own value
template <int CTRL, int ROWS>
__device__ inline unsigned long long dpp_u64(unsigned long long v)
{
    const int lo = (int)(unsigned)v, hi = (int)(unsigned)(v >> 32);
    const int l = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
    const int h = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false);
    return ((unsigned long long)(unsigned)h << 32) | (unsigned)l;
}

__device__ inline unsigned long long umax64(unsigned long long a, unsigned long long b) { return a > b ? a : b; }

// maximum of a 64-bit unsigned value over the wave (all 64 lanes active),
// returned in every lane: within each row of 16 lanes by quad permutes and
// mirrors, then across rows by the row broadcasts, read back from lane 63
__device__ inline unsigned long long wave_umax64(unsigned long long v)
{
    v = umax64(v, dpp_u64<0xB1, 0xF>(v));   // quad_perm [1,0,3,2]
    v = umax64(v, dpp_u64<0x4E, 0xF>(v));   // quad_perm [2,3,0,1]
    v = umax64(v, dpp_u64<0x141, 0xF>(v));  // row_half_mirror
    v = umax64(v, dpp_u64<0x140, 0xF>(v));  // row_mirror: row maximum in every lane
    v = umax64(v, dpp_u64<0x142, 0xA>(v));  // row_bcast:15 into rows 1 and 3
    v = umax64(v, dpp_u64<0x143, 0xC>(v));  // row_bcast:31 into rows 2 and 3
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return ((unsigned long long)hi << 32) | lo;
}

// Packed lines: x-sweeps of 2D and 3D grids whose lines the tiles fit badly.
// The n + 1 faces of every line follow one another in one sequence, line after
// line, and a workgroup takes 256 consecutive ones, the last of which is the
// first of the next workgroup; the cells with both faces in a workgroup are
// updated there.  Each line's part of a workgroup (at most PACK_SEGS parts)
// has its own halo nodes in LDS.  A tile per line computes 288 faces for 257
// where n = 256 and 1088 for 1025 where n = 1024; the sequence computes 258
// and 1029.
constexpr int PACK_MIN = 31, PACK_SEGS = 9;

// line of position a in a sequence of lines of b positions, the first of
// which a block's few hundred positions begin in: a / b, by comparison where
// they reach no further than the third line
__device__ inline int part_of(int a, int b)
{
    if (b > 150) return (a >= b) + (a >= 2 * b);
    int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
    q -= q * b > a;
    q += (q + 1) * b <= a;
    return q;
}

// Tile: BS face threads along the sweep direction (BS-1 cells), BA threads
// across it.  DIR == 0: blockDim = (BS, BA), across = y, blockIdx.z = z.
// DIR == 1: blockDim = (BA, BS), across = x, blockIdx.z = z.
// DIR == 2: blockDim = (BA, BS), across = x, blockIdx.z = y.
// The tile index along the sweep is blockIdx.y (in 2D and 3D), so that
// tiles sharing a halo have linear block indices gridDim.x apart: on the
// same XCD (and L2) when gridDim.x is a multiple of 8, and dispatched close
// together; 1D keeps the tiles on blockIdx.x, the dimension with room for
// long lines.
// The register budget of the sweeps is cut to three waves per SIMD (168
// VGPRs): the third wave hides more LDS and memory latency than the spills
// it causes cost (1024 x 512 step 0.441 -> 0.400 ms, 256^3 FP64 +3 %, FP32
// +11 %).  A fourth wave (128 VGPRs) pays for the plain FP64 sweeps once the
// face keeps few values past the flux limiter's check, where the
// workgroups' LDS fits: 1024 x 512 step -1.9 %, 256^3 x-sweep -1.5 %,
// z-sweep (three arrays read per cell after its barriers) -5 %, y-sweep
// -2 %.  In float a fourth wave does not pay (256^3 x-sweep +3.5 %), and a
// fifth (96 VGPRs) in 2D makes the 1024 x 512 step 14 % slower.
template <int D, int DIR, typename R, int WT>
constexpr int sweep_waves()
{
    return WT == 2 || (sizeof(R) == sizeof(double) && WT == 0 && D >= 2) ? 4 : 3;
}

// WT: 0 App. C weights, 1 learned weights, 2 the first-order schemes in double
// (the five-equation one and the four-equation HRM), a small kernel that
// stages one node beyond each end instead of three.
// WS: the launch is a stage update that also folds the wavespeed maxima of
// its output into A.wpart; a separate instantiation, so that the other
// launches keep their register allocation
template <int N, int D, int DIR, int BS, int BA, typename R, int WT, bool WS = false>
__global__ void __launch_bounds__(BS* BA, (sweep_waves<D, DIR, R, WT>())) k_sweep(const SweepArgs A)
{
    using F = NodeFields<N, D>;
    constexpr int M = 2 * N + D, IA = N + D + 1;
    constexpr int NA = N > 1 ? N - 1 : 1;
    constexpr int H = WT == 2 ? 1 : 3;  // nodes staged beyond the first and last face's cells
    // packed lines (x-sweeps in 2D and 3D, see the tiles above)
    constexpr bool PK = D >= 2 && DIR == 0 && BA == 1;
    constexpr int LN = BS - 1 + 2 * H;
    constexpr int T = BS * BA, NQ = PK ? T + (2 * H - 1) * PACK_SEGS : LN * BA;
    constexpr int FS = NQ;
    constexpr int NS = DIR == 0 ? 1 : BA;
    static_assert((BS * BA) % 64 == 0, "whole waves");
    __shared__ double lds[F::COUNT * FS];

    const int ts = DIR == 0 ? threadIdx.x : threadIdx.y;
    const int ta = DIR == 0 ? threadIdx.y : threadIdx.x;
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    const long long st[3] = {1, A.n[0], (long long)A.n[0] * A.n[1]};
    int c0, abase, other, adim, odim;
    if (DIR == 0) {
        c0 = (D == 1 ? blockIdx.x : blockIdx.y) * (BS - 1);
        abase = (D == 1 ? blockIdx.y : blockIdx.x) * BA;
        other = blockIdx.z;
        adim = 1;
        odim = 2;
    } else if (DIR == 1) {
        c0 = blockIdx.y * (BS - 1);
        abase = blockIdx.x * BA;
        other = blockIdx.z;
        adim = 0;
        odim = 2;
    } else {
        c0 = blockIdx.y * (BS - 1);
        abase = blockIdx.x * BA;
        other = blockIdx.z;
        adim = 0;
        odim = 1;
    }
    const int nsw = A.n[DIR], na = A.n[adim];
    const long long nc = A.ncell;
    // packed lines: the block's first face is face p0 of line line0; thread t
    // has face p0 + t - seg (n + 1) of line line0 + seg
    [[maybe_unused]] long long nlines = 0, line0 = 0, line = 0;
    [[maybe_unused]] int p0 = 0, seg = 0, lastseg = 0, face = 0;
    if constexpr (PK) {
        const int np = nsw + 1;
        nlines = (long long)A.n[1] * A.n[2];
        // blocks are dealt to the eight XCDs in turn; each takes one contiguous
        // eighth of the sequence, whose shared halos then meet in its L2
        // (1024 x 512 step -1.6 %)
        const unsigned nb = gridDim.x, xcd = blockIdx.x & 7u;
        const unsigned bx = xcd * (nb >> 3) + min(xcd, nb & 7u) + (blockIdx.x >> 3);
        if (A.rnp) {
            // fewer than 2^32 faces: the line by a scalar multiplication
            const unsigned g0 = bx * (BS - 1u);
            unsigned l0 = __umulhi(g0, A.rnp);
            p0 = (int)(g0 - l0 * np);
            while (p0 >= np) {
                p0 -= np;
                ++l0;
            }
            line0 = l0;
        } else {
            const long long g0 = (long long)bx * (BS - 1);
            line0 = g0 / np;
            p0 = (int)(g0 - line0 * np);
        }
        seg = part_of(p0 + ts, np);
        lastseg = part_of(p0 + BS - 1, np);
        face = p0 + ts - seg * np;
        line = line0 + seg;
    }
    auto base = [](int a, int l) { return DIR == 0 ? a * LN + l : l * BA + a; };

    // stage the node tile (sweep index c0-H .. c0+BS-2+H) with its primitives.
    // The staging waves run at raised priority, so that a workgroup starting
    // beside others still computing faces gets its loads out first (1024 x
    // 512 step -2.4 %, 256^3 FP64 -1 %, FP32 -2.6 %; raising it also around
    // the stage update's loads measured slower).  A tile has a few more nodes
    // than threads: the loads of a thread's second node are issued with those
    // of its first, so that the waves that have one wait for memory once.
    __builtin_amdgcn_s_setprio(3);
    {
        // (in float one node at a time: the registers of the second cost more)
        constexpr int IT = (NQ + T - 1) / T, LOADS = sizeof(R) == sizeof(double) ? IT : 1;
        double W[LOADS][M];
        auto load = [&](int q, double* w) {
            const double* src = A.Ws;
            long long idx, stride = nc;
            int gi;
            long long line;  // index of the node's line among the lines along x (packed lines only)
            if constexpr (PK) {
                const int pos = p0 + q, seg = part_of(pos, A.n[0] + 1 + 2 * H - 1);
                gi = pos - seg * (A.n[0] + 2 * H) - H;
                line = line0 + seg < nlines ? line0 + seg : nlines - 1;
            } else {
                gi = c0 - H + (DIR == 0 ? q % LN : q / BA);
            }
            const int ca = min(abase + (DIR == 0 ? q / LN : q % BA), na - 1);
            if ((gi < 0 && A.bclo == BC_DIRICHLET) || (gi >= nsw && A.bchi == BC_DIRICHLET)) {
                // Dirichlet: every ghost node takes the boundary state of its line
                src = gi < 0 ? A.blo : A.bhi;
                if constexpr (PK) {
                    idx = line;
                    stride = nlines;
                } else {
                    idx = ca + (long long)na * other;
                    stride = (long long)na * A.n[odim];
                }
            } else {
                const int g = map_bc(gi, nsw, A.bclo, A.bchi);
                if constexpr (PK)
                    idx = line * A.n[0] + g;
                else
                    idx = g * st[DIR] + ca * st[adim] + other * st[odim];
            }
#pragma unroll
            for (int c = 0; c < M; ++c) w[c] = src[c * stride + idx];
        };
        auto store = [&](int q, const double* w) {
            const EosDev e = kload<EosDev>(kernel_args() + offsetof(SweepArgs, e));
            St<N, D> s;
            state_from_W<N, D>(e, w, s);
            if constexpr (WT == 2)
                if (A.P.flags & F_FOUR_EQ) hrm4_pc<N, D>(e, s, s.p, s.c);
            const int b = PK ? q : base(DIR == 0 ? q / LN : q % BA, DIR == 0 ? q % LN : q / BA);
#pragma unroll
            for (int c = 0; c < M; ++c) lds[c * FS + b] = w[c];
#pragma unroll
            for (int d = 0; d < D; ++d) lds[(F::U + d) * FS + b] = s.u[d];
            lds[F::P * FS + b] = s.p;
            lds[F::RHO * FS + b] = s.rho;
            lds[F::C * FS + b] = s.c;
        };
        const int nq = PK ? T + (2 * H - 1) * (lastseg + 1) : NQ;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int q = tid + it * T;
            if ((it + 1) * T > NQ && q >= nq) continue;
            load(q, W[LOADS > 1 ? it : 0]);
            if constexpr (LOADS == 1) store(q, W[0]);
        }
        if constexpr (LOADS > 1)
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int q = tid + it * T;
                if ((it + 1) * T > NQ && q >= nq) continue;
                store(q, W[it]);
            }
    }
    __builtin_amdgcn_s_setprio(0);
    // On a line every sweep spans all of it, so the step's first sweep takes
    // the maximum of the wavespeed partials itself, every workgroup the same
    // one, and forms the time step that it works with; its first workgroup
    // leaves it for the later sweeps.  The second sweep's first workgroup, when
    // nobody reads them any more, advances the device time and clears the
    // partials for the third to fold into.  That saves the launch of
    // k_reduce_dt, a fifth of a short first-order step.
    double dt_step = 0.0, lam = 0.0;
    if constexpr (D == 1) {
        __shared__ double shm[T / 64];
        if (A.phase == 1) {
            double m = 0.0;
            for (int i = tid; i < A.npart; i += T) m = nmax(m, A.part[i]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) m = nmax(m, __shfl_xor(m, off, 64));
            if ((tid & 63) == 0) shm[tid >> 6] = m;
        }
        __syncthreads();
        if (A.phase == 1) {
            double m = shm[0], slot[5] = {0.0, 0.0, 0.0, 0.0, A.slot[4]};
#pragma unroll
            for (int i = 1; i < T / 64; ++i) m = nmax(m, shm[i]);
            dt_from_max(&m, A.dt, slot);
            dt_step = slot[0];
            lam = slot[1];
            if (tid == 0 && blockIdx.x == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) A.slotw[i] = slot[i];
                *A.tnext = slot[4];
            }
        } else {
            dt_step = A.slot[0];
            lam = A.slot[1];
            if (A.phase == 2 && blockIdx.x == 0) {
                for (int i = tid; i < (int)A.nslot; i += T) A.part[i] = 0.0;
                if (tid == 0) A.slotw[4] = *A.tnext;
            }
        }
    } else {
        __syncthreads();
        lam = A.slot[1 + DIR];
    }

    // one face per thread: between sweep nodes c0-1+ts and c0+ts.  In the
    // z-sweep a wave holds four consecutive ts; one whose faces all lie
    // beyond face nsw (three waves of the last tile of a 256-cell line)
    // skips them and their LDS writes, which no cell reads (256^3 z-sweep
    // -1.3 %; the same skip in the y-sweeps and in 1D measured no better,
    // the branch costing them as much in register allocation)
    const bool live = DIR != 2 || c0 + __builtin_amdgcn_readfirstlane(tid >> 6) * (64 / BA) <= nsw;
    unsigned cnt = 0;  // packed counts (cnt_one)
    double G[M], Gp[NA];
    if (live) {
        unsigned lc = 0;
        const KArg ka = kernel_args();
        // the first-order float scheme is the general kernel's
        constexpr int LOW = WT == 2 ? 2 : (sizeof(R) == sizeof(double) ? 0 : 1);
        face_flux<N, D, DIR, NS, FS, R, WT == 1 ? 1 : 0, LOW>(
            lds + (PK ? ts + (2 * H - 1) * seg + H - 3 : base(ta, ts + H - 3)), ka + offsetof(SweepArgs, e), ka + offsetof(SweepArgs, P), lam, G, Gp, lc);
        // face c0+ts is counted once: the last face of a tile is the first
        // face of the next tile unless it is the boundary face nsw
        bool ok;
        if constexpr (PK) {
            ok = line < nlines && (ts < BS - 1 || (face == nsw && line == nlines - 1));
        } else {
            const int f = c0 + ts;
            ok = f <= nsw && (ts < BS - 1 || f == nsw) && (abase + ta < na);
        }
        if (ok) cnt = lc;
    }
    // A middle direction only adds to the right-hand side (MODE_ADD): its
    // cell's accumulated values are loaded here, before the barriers, so that
    // their latency overlaps the wait for the block's slowest face (3D
    // y-sweep -11 %; the other directions keep their loads where they are
    // used, which measured faster for them)
    constexpr bool MID = DIR > 0 && DIR < D - 1;
    double Rc[MID ? M : 1];
    if constexpr (MID) {
        const int ci = c0 + ts, ca = abase + ta;
        if (ts < BS - 1 && ci < nsw && ca < na) {
            const long long cell = ci * st[DIR] + ca * st[adim] + other * st[odim];
#pragma unroll
            for (int c = 0; c < M; ++c) Rc[c] = A.rhs[c * nc + cell];
        }
    }
    __syncthreads();
    if (live) {
        const int b = PK ? ts : base(ta, ts);
#pragma unroll
        for (int c = 0; c < M; ++c) lds[c * FS + b] = G[c];
#pragma unroll
        for (int k = 0; k < N - 1; ++k) lds[(M + k) * FS + b] = Gp[k];
    }
    __syncthreads();

    // flux difference of cell c0+ts: faces ts (i-1/2) and ts+1 (i+1/2)
    const int ci = PK ? face : c0 + ts, ca = abase + ta;
    double wmax[D];
#pragma unroll
    for (int d = 0; d < D; ++d) wmax[d] = 0.0;
    if (ts < BS - 1 && ci < nsw && (PK ? line < nlines : ca < na)) {
        const long long cell = PK ? line * nsw + ci : ci * st[DIR] + ca * st[adim] + other * st[odim];
        const int bl = PK ? ts : base(ta, ts), br = PK ? ts + 1 : base(ta, ts + 1);
        double L[M];
#pragma unroll
        for (int c = 0; c < IA; ++c) L[c] = flux_difference(lds[c * FS + br], lds[c * FS + bl], A.idx);
#pragma unroll
        for (int k = 0; k < N - 1; ++k)
            L[IA + k] = flux_difference(lds[(IA + k) * FS + br], lds[(M + k) * FS + bl], A.idx);
        if (A.mode == MODE_WRITE) {
#pragma unroll
            for (int c = 0; c < M; ++c) A.rhs[c * nc + cell] = L[c];
        } else if (A.mode == MODE_ADD) {
            if constexpr (MID) {
#pragma unroll
                for (int c = 0; c < M; ++c) A.rhs[c * nc + cell] = add_direction(Rc[c], L[c]);
            } else {
#pragma unroll
                for (int c = 0; c < M; ++c) A.rhs[c * nc + cell] = add_direction(A.rhs[c * nc + cell], L[c]);
            }
        } else {
            const double dt = D == 1 ? dt_step : A.slot[0];
            double w[M];
            if (__builtin_expect(A.hold && dt == 0.0, 0)) {
                // every stage of a step of length 0 is W^n in exact arithmetic;
                // written as such, a run held at its end time stays bit for bit
#pragma unroll
                for (int c = 0; c < M; ++c) w[c] = A.Wn[c * nc + cell];
            } else {
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    const double Lc = D > 1 ? add_direction(A.rhs[c * nc + cell], L[c]) : L[c];
                    w[c] = stage_value(A.a, A.b, A.Wn[c * nc + cell], A.Ws[c * nc + cell], dt, Lc);
                }
                if (A.relax && !relax_cell<N, D>(kload<EosDev>(kernel_args() + offsetof(SweepArgs, e)), w))
                    cnt += cnt_one(C_RELAX_BAD);
            }
#pragma unroll
            for (int c = 0; c < M; ++c) A.Wout[c * nc + cell] = w[c];
            if constexpr (WS) {
                // Sec. 4.1.2: |u_d| + c of the new state, for the next time step
                const EosDev e = kload<EosDev>(kernel_args() + offsetof(SweepArgs, e));
                St<N, D> s;
                state_from_W<N, D>(e, w, s);
                double cs = s.c;
                if constexpr (WT == 2)
                    if (A.P.flags & F_FOUR_EQ) {
                        double p;
                        hrm4_pc<N, D>(e, s, p, cs);
                    }
#pragma unroll
                for (int d = 0; d < D; ++d) wmax[d] = fabs(s.u[d]) + cs;
            }
        }
    }
    if constexpr (WS) {
        // wave maximum, folded into slot (linear block index) % nslot, which
        // the time-step reduction has cleared.  The values are +0 or above,
        // or NaN; their bit patterns order as unsigned integers the same way,
        // with every NaN above every number, so the maximum is taken on the
        // bits: without branches, and by the 64-bit unsigned atomic max.  Each
        // wave folds its own maximum (no block barrier: a wave leaves as soon
        // as its atomics are issued, and the next block's tile starts sooner)
        unsigned long long wb[D];
#pragma unroll
        for (int d = 0; d < D; ++d) wb[d] = wave_umax64((unsigned long long)__double_as_longlong(wmax[d]));
        if ((tid & 63) == 0) {
            const unsigned blk = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
            unsigned long long* slot = (unsigned long long*)A.wpart + (blk & (A.nslot - 1u)) * D;
#pragma unroll
            for (int d = 0; d < D; ++d) atomicMax(slot + d, wb[d]);
        }
    }
    flush_counters(cnt, A.cnt);
}

// A stage of a small 2D grid, both directions of a tile of 15 x 7 cells in one
// launch: waves 0 and 1 take its 16 x 7 faces along x, waves 2 and 3 its 15 x 8
// along y, and the cells add both differences in the order of the two sweeps
// (the same bits).  A sweep of such a grid is bound by the latency of one wave
// of faces on a SIMD and by its launch, and this takes one of each instead of
// two and no pass through the right-hand side (127 x 65, two species, a stage
// 19.3 -> 10.7 us); the tile computes 2.21 faces a cell and stages 2.26 nodes, so
// larger grids, which are bound by issue, are left to the sweeps.
struct PlaneArgs {
    SweepArgs s;  // first: its members are read through the argument pointer; x sides
    int bclo, bchi;
    const double* blo;
    const double* bhi;
    double idx;
};
constexpr int PLANE_X = 15, PLANE_Y = 7;

template <int N, typename R>
__global__ void __launch_bounds__(256, 2) k_plane(const PlaneArgs A)
{
    using F = NodeFields<N, 2>;
    constexpr int D = 2, M = 2 * N + D, IA = N + D + 1;
    constexpr int NA = N > 1 ? N - 1 : 1;
    constexpr int LX = PLANE_X + 6, FS = LX * (PLANE_Y + 6), XF = 128;  // the y faces' slots start at XF
    static_assert(PLANE_X + 1 == 16 && 16 * PLANE_Y <= XF && PLANE_X * (PLANE_Y + 1) <= 256 - XF && FS >= 256, "tile");
    // the node tile without its corners: halo rows of PLANE_X nodes, whole rows of LX
    constexpr int HALO = 3 * PLANE_X, ROWS = LX * PLANE_Y;
    static_assert(2 * HALO + ROWS <= 256, "one node a thread");
    __shared__ double lds[F::COUNT * FS];
    const int tid = threadIdx.x;
    const int n0 = A.s.n[0], n1 = A.s.n[1], x0 = blockIdx.x * PLANE_X, y0 = blockIdx.y * PLANE_Y;
    const int nx = min(PLANE_X, n0 - x0), ny = min(PLANE_Y, n1 - y0);  // cells of the tile
    const long long nc = A.s.ncell;

    if (tid < 2 * HALO + ROWS) {
        int lx, ly;
        if (tid < HALO) {
            ly = tid / PLANE_X;
            lx = 3 + tid % PLANE_X;
        } else if (tid < HALO + ROWS) {
            ly = 3 + (tid - HALO) / LX;
            lx = (tid - HALO) % LX;
        } else {
            ly = 3 + PLANE_Y + (tid - HALO - ROWS) / PLANE_X;
            lx = 3 + (tid - HALO - ROWS) % PLANE_X;
        }
        const int gx = x0 - 3 + lx, gy = y0 - 3 + ly;
        const int cx = map_bc(gx, n0, A.s.bclo, A.s.bchi), cy = map_bc(gy, n1, A.bclo, A.bchi);
        const double* src = A.s.Ws;
        long long idx = (long long)cy * n0 + cx, stride = nc;
        // Dirichlet: every ghost node takes the boundary state of its line
        if ((gx < 0 && A.s.bclo == BC_DIRICHLET) || (gx >= n0 && A.s.bchi == BC_DIRICHLET)) {
            src = gx < 0 ? A.s.blo : A.s.bhi;
            idx = cy;
            stride = n1;
        } else if ((gy < 0 && A.bclo == BC_DIRICHLET) || (gy >= n1 && A.bchi == BC_DIRICHLET)) {
            src = gy < 0 ? A.blo : A.bhi;
            idx = cx;
            stride = n0;
        }
        double w[M];
#pragma unroll
        for (int c = 0; c < M; ++c) w[c] = src[c * stride + idx];
        const EosDev e = kload<EosDev>(kernel_args() + offsetof(SweepArgs, e));
        St<N, D> s;
        state_from_W<N, D>(e, w, s);
        const int b = ly * LX + lx;
#pragma unroll
        for (int c = 0; c < M; ++c) lds[c * FS + b] = w[c];
#pragma unroll
        for (int d = 0; d < D; ++d) lds[(F::U + d) * FS + b] = s.u[d];
        lds[F::P * FS + b] = s.p;
        lds[F::RHO * FS + b] = s.rho;
        lds[F::C * FS + b] = s.c;
    }
    __syncthreads();

    // faces; lanes without one repeat the last of their direction, and a face
    // between two tiles is counted by the upper one
    double G[M], Gp[NA];
    unsigned cnt = 0, lc = 0;
    constexpr int LOW = sizeof(R) == sizeof(double) ? 0 : 1;
    if (__builtin_amdgcn_readfirstlane(tid) < XF) {
        const int fx = tid % 16, fy = tid / 16, qx = min(fx, nx), qy = min(fy, ny - 1);
        face_flux<N, D, 0, 1, FS, R, 0, LOW>(lds + (qy + 3) * LX + qx, kernel_args() + offsetof(SweepArgs, e),
                                             kernel_args() + offsetof(SweepArgs, P), A.s.slot[1], G, Gp, lc);
        if (fy < ny && (fx < nx || x0 + fx == n0) && (fx < PLANE_X || x0 + fx == n0)) cnt = lc;
    } else {
        const int f = tid - XF, fx = f % PLANE_X, fy = f / PLANE_X, qx = min(fx, nx - 1), qy = min(fy, ny);
        face_flux<N, D, 1, LX, FS, R, 0, LOW>(lds + qy * LX + qx + 3, kernel_args() + offsetof(SweepArgs, e),
                                              kernel_args() + offsetof(SweepArgs, P), A.s.slot[2], G, Gp, lc);
        if (fx < nx && fy <= PLANE_Y && (fy < ny || y0 + fy == n1) && (fy < PLANE_Y || y0 + fy == n1)) cnt = lc;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < M; ++c) lds[c * FS + tid] = G[c];
#pragma unroll
    for (int k = 0; k < N - 1; ++k) lds[(M + k) * FS + tid] = Gp[k];
    __syncthreads();

    const int ci = tid % PLANE_X, cj = tid / PLANE_X;
    double wmax[D] = {0.0, 0.0};
    if (ci < nx && cj < ny) {
        const long long cell = (long long)(y0 + cj) * n0 + x0 + ci;
        const int bx = cj * 16 + ci, by = XF + cj * PLANE_X + ci;
        const double dt = A.s.slot[0];
        double w[M];
        if (__builtin_expect(A.s.hold && dt == 0.0, 0)) {
#pragma unroll
            for (int c = 0; c < M; ++c) w[c] = A.s.Wn[c * nc + cell];
        } else {
#pragma unroll
            for (int c = 0; c < M; ++c) {
                const int m = c >= IA ? M + c - IA : c;  // the pair's slots of the volume fractions
                const double Lx = flux_difference(lds[c * FS + bx + 1], lds[m * FS + bx], A.s.idx);
                const double Ly = flux_difference(lds[c * FS + by + PLANE_X], lds[m * FS + by], A.idx);
                w[c] = stage_value(A.s.a, A.s.b, A.s.Wn[c * nc + cell], A.s.Ws[c * nc + cell], dt, add_direction(Lx, Ly));
            }
            if (A.s.relax && !relax_cell<N, D>(kload<EosDev>(kernel_args() + offsetof(SweepArgs, e)), w)) cnt += cnt_one(C_RELAX_BAD);
        }
#pragma unroll
        for (int c = 0; c < M; ++c) A.s.Wout[c * nc + cell] = w[c];
        if (A.s.wpart) {
            St<N, D> s;
            state_from_W<N, D>(kload<EosDev>(kernel_args() + offsetof(SweepArgs, e)), w, s);
#pragma unroll
            for (int d = 0; d < D; ++d) wmax[d] = fabs(s.u[d]) + s.c;
        }
    }
    if (A.s.wpart) {
        unsigned long long wb[D];
#pragma unroll
        for (int d = 0; d < D; ++d) wb[d] = wave_umax64((unsigned long long)__double_as_longlong(wmax[d]));
        if ((tid & 63) == 0) {
            const unsigned blk = blockIdx.x + gridDim.x * blockIdx.y;
            unsigned long long* slot = (unsigned long long*)A.s.wpart + (blk & (A.s.nslot - 1u)) * D;
#pragma unroll
            for (int d = 0; d < D; ++d) atomicMax(slot + d, wb[d]);
        }
    }
    flush_counters(cnt, A.s.cnt);
}

// The pointwise kernels are bound by memory.  V cells per thread: two, with
// 16-byte loads and stores, where every plane of every array is aligned for
// them (an even number of cells and 16-byte pointers), else one.
template <int V>
__device__ inline void load_cells(const double* p, double* v)
{
    if constexpr (V == 2) {
        const double2 t = *(const double2*)p;
        v[0] = t.x;
        v[1] = t.y;
    } else {
        v[0] = *p;
    }
}
template <int V>
__device__ inline void store_cells(double* p, const double* v)
{
    if constexpr (V == 2)
        *(double2*)p = make_double2(v[0], v[1]);
    else
        *p = v[0];
}

template <int N, int D, int V>
__global__ void __launch_bounds__(256) k_relax(double* W, long long nc, EosDev e, unsigned long long* cnt)
{
    constexpr int M = 2 * N + D, IA = N + D + 1;
    unsigned c[C_N] = {0, 0, 0, 0, 0, 0, 0};
    for (long long i = (blockIdx.x * 256ll + threadIdx.x) * V; i < nc; i += (long long)gridDim.x * 256 * V) {
        double x[IA][V], al[N - 1][V];
#pragma unroll
        for (int k = 0; k < IA; ++k) load_cells<V>(W + k * nc + i, x[k]);
        bool bad = false;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            double w[M];
#pragma unroll
            for (int k = 0; k < IA; ++k) w[k] = x[k][j];
            if (relax_cell<N, D>(e, w)) {
#pragma unroll
                for (int k = 0; k < N - 1; ++k) al[k][j] = w[IA + k];
            } else {
                // left unchanged
                c[C_RELAX_BAD]++;
                bad = true;
#pragma unroll
                for (int k = 0; k < N - 1; ++k) al[k][j] = W[(IA + k) * nc + i + j];
            }
        }
        if (V == 1 && bad) continue;
#pragma unroll
        for (int k = 0; k < N - 1; ++k) store_cells<V>(W + (IA + k) * nc + i, al[k]);
    }
    flush_counters(c, cnt);
}

// Sec. 3: p*, T* (eq:p_relax, eq:T_relax_e) and the sound speed of the
// four-equation HRM (eq:4_eqn_sos) of every cell; NaN where the state has
// no admissible relaxed state.  Null outputs are skipped.  p* and T* are
// evaluated once for all outputs (2048 x 1280, two species: 36 -> 27.7 us);
// the kernel is now bound by memory: 168 MB in that time, 6.1 TB/s.
template <int N, int D, int V>
__global__ void __launch_bounds__(256) k_equilibrium(const double* W, long long nc, EosDev e, double* p_out,
                                                      double* T_out, double* c_out)
{
    constexpr int IA = N + D + 1;
    for (long long i = (blockIdx.x * 256ll + threadIdx.x) * V; i < nc; i += (long long)gridDim.x * 256 * V) {
        double x[IA][V], p[V], T[V], c[V];
#pragma unroll
        for (int k = 0; k < IA; ++k) load_cells<V>(W + k * nc + i, x[k]);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            double w[IA];
#pragma unroll
            for (int k = 0; k < IA; ++k) w[k] = x[k][j];
            p[j] = T[j] = c[j] = __builtin_nan("");
            double pj, Tj;
            if (relaxed_pT<N, D>(e, w, pj, Tj)) {
                St<N, D> s;
#pragma unroll
                for (int k = 0; k < N; ++k) s.ar[k] = w[k];
#pragma unroll
                for (int d = 0; d < D; ++d) s.mom[d] = w[N + d];
                s.E = w[N + D];
                p[j] = pj;
                T[j] = Tj;
                c[j] = hrm4_c<N, D>(e, s, pj);
            }
        }
        if (p_out) store_cells<V>(p_out + i, p);
        if (T_out) store_cells<V>(T_out + i, T);
        if (c_out) store_cells<V>(c_out + i, c);
    }
}

// only >= 0: the other directions' maxima are 0 (Dirichlet ghost states
// count for the direction normal to their face only)
template <int N, int D, int V>
__global__ void __launch_bounds__(256) k_wavespeed(const double* W, long long nc, EosDev e, int four, int only,
                                                    double* part)
{
    constexpr int M = 2 * N + D;
    __shared__ double sh[4 * 3];
    double m[D];
#pragma unroll
    for (int d = 0; d < D; ++d) m[d] = 0.0;
    for (long long i = (blockIdx.x * 256ll + threadIdx.x) * V; i < nc; i += (long long)gridDim.x * 256 * V) {
        double x[M][V];
#pragma unroll
        for (int k = 0; k < M; ++k) load_cells<V>(W + k * nc + i, x[k]);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            double w[M];
#pragma unroll
            for (int k = 0; k < M; ++k) w[k] = x[k][j];
            St<N, D> s;
            state_from_W<N, D>(e, w, s);
            double c = s.c;
            if (four) {  // the four-equation model solved directly: its own sound speed
                double p;
                hrm4_pc<N, D>(e, s, p, c);
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (only < 0 || only == d) m[d] = nmax(m[d], fabs(s.u[d]) + c);
        }
    }
    block_max<D>(m, sh);
    if (threadIdx.x == 0)
#pragma unroll
        for (int d = 0; d < D; ++d) part[blockIdx.x * D + d] = m[d];
}

// threads of the one-block reductions of the partials
constexpr int RT = 256;

// this thread's share of the maximum of nb partials (one block of RT
// threads): eight loads in flight per pass instead of one
template <int D>
__device__ inline void partial_max(const double* part, int nb, double* m)
{
    for (int i0 = threadIdx.x; i0 < nb; i0 += RT * 8) {
        double v[8][D];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int d = 0; d < D; ++d) v[u][d] = i0 + RT * u < nb ? part[(i0 + RT * u) * D + d] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int d = 0; d < D; ++d) m[d] = nmax(m[d], v[u][d]);
    }
}

template <int D>
__global__ void __launch_bounds__(RT) k_reduce_max(const double* part, int nb, double* out)
{
    __shared__ double sh[(RT / 64) * 3];
    double m[D];
#pragma unroll
    for (int d = 0; d < D; ++d) m[d] = 0.0;
    partial_max<D>(part, nb, m);
    block_max<D>(m, sh);
    if (threadIdx.x == 0)
#pragma unroll
        for (int d = 0; d < D; ++d) out[d] = m[d];
}

__global__ void k_dt(const double* maxs, DtArgs a, double* slot)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) dt_from_max(maxs, a, slot);
}

// grid-wide maximum of the wavespeed partials and the time step, one block;
// then the first nclear partials (the slots the last sweep of the step folds
// into) are set to +0, each by the thread that read it
template <int D>
__global__ void __launch_bounds__(RT) k_reduce_dt(double* part, int nb, int nclear, double* maxs, DtArgs a,
                                                   double* slot)
{
    __shared__ double sh[(RT / 64) * 3];
    double m[D];
#pragma unroll
    for (int d = 0; d < D; ++d) m[d] = 0.0;
    partial_max<D>(part, nb, m);
    for (int i = threadIdx.x; i < nclear; i += RT)
#pragma unroll
        for (int d = 0; d < D; ++d) part[i * D + d] = 0.0;
    block_max<D>(m, sh);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) maxs[d] = m[d];
        dt_from_max(maxs, a, slot);
    }
}

// learned interpolation of n stencils U[i][0..4] (one lane per stencil; the
// whole wave evaluates the network together)
__global__ void __launch_bounds__(64) k_mlp_infer(const MlpPacked* m, const double* U, long long n, double eps,
                                                  double* val, float* om)
{
    const long long i = (long long)blockIdx.x * 64 + threadIdx.x;
    double u[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (i < n)
#pragma unroll
        for (int j = 0; j < 5; ++j) u[j] = U[i * 5 + j];
    float x[5], z[3], w[3];
    mlp_inputs(u, x);
    mlp_logits(m, x, z);
    const bool ok = mlp_omega(z, x, w);
    if (i < n) {
        val[i] = ok ? mlp_value(u, w) : weno_is(u[0], u[1], u[2], u[3], u[4], eps);
#pragma unroll
        for (int k = 0; k < 3; ++k) om[i * 3 + k] = w[k];
    }
}

__global__ void k_zero_u64(unsigned long long* p, int n)
{
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

}  // namespace hrm

// ------------------------------------------------------------------ context
struct hrm_ctx {
    int N, D, M;
    int n[3];
    double dx[3];
    int bclo[3], bchi[3];
    int precision, weights, flags;
    long long ncell;
    hrm::EosDev eos;
    hrm::ParDev par;
    double* d_rhs;
    double* d_W1;
    double* d_W2;
    double* d_part;
    int npart;               // wavespeed partial blocks of hrm_max_wavespeed
    int nslot;               // partial slots the last sweep of a step folds its blocks into
    double* d_maxs;
    unsigned long long* d_cnt;
    double* d_bnd[3][2];     // Dirichlet ghost states per face (M x face cells), null elsewhere
    int bnd_set[3][2];
    long long nface[3];      // cells of a face normal to each dimension
    int nbpart[3];           // wavespeed partial blocks per Dirichlet face of that dimension
    hrm::MlpPacked* d_mlp;  // learned weights (HRM_WEIGHTS_MLP)
    int mlp_ready;
    hipStream_t last_stream;
    // hrm_step replay: one captured RK3 step per argument set
    hipStream_t cap_stream;
    hipGraphExec_t gexec;
    double* g_W;
    double* g_slot;
    double g_cfl, g_dt_fixed, g_t_end;
    // opt-in event timing
    int timing_mask;
    int npending;
    int pend_kind[4096];
    hipEvent_t pend_ev[4096][2];
    hipEvent_t pool[4096][2];
    int pool_ready;
    double tms[HRM_NTIMERS];
    long long tcnt[HRM_NTIMERS];
    char err[512];
};

namespace {

int fail(hrm_ctx* c, int code, const char* fmt, const char* a = "", long long v = 0)
{
    if (c) snprintf(c->err, sizeof(c->err), fmt, a, v);
    return code;
}

int check_launch(hrm_ctx* c, const char* what)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        snprintf(c->err, sizeof(c->err), "%s: %s", what, hipGetErrorString(e));
        return HRM_EDEVICE;
    }
    return HRM_OK;
}

void fold_timers(hrm_ctx* c)
{
    for (int i = 0; i < c->npending; ++i) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, c->pend_ev[i][0], c->pend_ev[i][1]) == hipSuccess) {
            c->tms[c->pend_kind[i]] += ms;
            c->tcnt[c->pend_kind[i]] += 1;
        }
    }
    c->npending = 0;
}

// records an event pair around the launches in its scope when `kind` is selected
struct TimerScope {
    hrm_ctx* c;
    int kind;
    hipStream_t s;
    int slot;
    TimerScope(hrm_ctx* c_, int kind_, hipStream_t s_) : c(c_), kind(kind_), s(s_), slot(-1)
    {
        if (!c->pool_ready || !((c->timing_mask >> kind) & 1)) return;
        if (c->npending == 4096) {
            (void)hipStreamSynchronize(s);
            fold_timers(c);
        }
        slot = c->npending++;
        c->pend_kind[slot] = kind;
        c->pend_ev[slot][0] = c->pool[slot][0];
        c->pend_ev[slot][1] = c->pool[slot][1];
        (void)hipEventRecord(c->pend_ev[slot][0], s);
    }
    ~TimerScope()
    {
        if (slot >= 0) (void)hipEventRecord(c->pend_ev[slot][1], s);
    }
};

// tile of the sweep in direction dir: BS face threads along it, BA across.
// A tile computes BS faces for BS - 1 cells, so a line of n cells takes
// ceil(n / (BS - 1)) tiles.  Along x (2D, 3D) the better of 64 x 4 and 32 x 8,
// unless the packed sequence of all lines (256 threads) needs 8 % fewer faces
// and fills the chip (1024 workgroups): it costs a few per cent in index
// arithmetic and straddled cache lines (256^3, 10 % fewer: step -1.9 %; 1024 x
// 512, 5 % fewer: +0.7 %; 1000 x 500, 2 % fewer: +2.3 %; 127 x 65, 20 % fewer
// but 33 workgroups: +1 to +5 %).
void sweep_tile(const hrm_ctx* c, int dir, int& BS, int& BA)
{
    const long long n = c->n[dir];
    BS = BA = 16;
    if (c->D == 1) {
        BS = 256;
        BA = 1;
    } else if (dir == 0) {
        const long long f64 = (n + 62) / 63 * 64, f32 = (n + 30) / 31 * 32;
        if (n >= hrm::PACK_MIN && 100 * std::min(f64, f32) > 108 * (n + 1) && (n + 1) * c->n[1] * c->n[2] > 1024 * 255) {
            BS = 256;
            BA = 1;
        } else {
            BS = f32 < f64 ? 32 : 64;
            BA = f32 < f64 ? 8 : 4;
        }
    }
}

dim3 sweep_grid(const hrm_ctx* c, int dir, int BS, int BA)
{
    const int cells = BS - 1;
    if (dir == 0 && c->D == 1) return dim3((c->n[0] + cells - 1) / cells, (c->n[1] + BA - 1) / BA, c->n[2]);
    if (dir == 0 && BA == 1) {
        const long long faces = (c->n[0] + 1ll) * c->n[1] * c->n[2];
        return dim3((unsigned)((faces - 1 + cells - 1) / cells));
    }
    if (dir == 0) return dim3((c->n[1] + BA - 1) / BA, (c->n[0] + cells - 1) / cells, c->n[2]);
    if (dir == 1) return dim3((c->n[0] + BA - 1) / BA, (c->n[1] + cells - 1) / cells, c->n[2]);
    return dim3((c->n[0] + BA - 1) / BA, (c->n[2] + cells - 1) / cells, c->n[1]);
}

// the sizes hrm_create takes: those of a launch with tiles of 63 cells along x
// and 15 along y and z, the other dimensions on the grid's z (y and z at most
// 65535 blocks)
bool sizes_fit(const hrm_ctx* c)
{
    const int most = 65535;
    if (c->D >= 2 && ((c->n[0] + 62ll) / 63 > most || (c->n[1] + 14ll) / 15 > most)) return false;
    return c->D < 3 || (c->n[1] <= most && c->n[2] <= most);
}

template <int N, int D>
struct Ops {
    static constexpr int M = 2 * N + D;

    template <int DIR, int BS, int BA>
    static void launch_dir(hrm_ctx* c, hrm::SweepArgs& A, hipStream_t s)
    {
        dim3 blk = DIR == 0 ? dim3(BS, BA) : dim3(BA, BS);
        const dim3 grd = sweep_grid(c, DIR, BS, BA);
        A.bclo = c->bclo[DIR];
        A.bchi = c->bchi[DIR];
        A.blo = c->d_bnd[DIR][0];
        A.bhi = c->d_bnd[DIR][1];
        A.idx = 1.0 / c->dx[DIR];
        if (DIR == 0) A.rnp = (c->n[0] + 1ll) * c->n[1] * c->n[2] < (1ll << 32) ? (unsigned)((1ll << 32) / (c->n[0] + 1)) : 0u;
        TimerScope t(c, HRM_T_SWEEP_X + DIR, s);
        if constexpr (DIR == D - 1) {
            if (A.wpart) {
                launch_kernel<DIR, BS, BA, true>(c, A, grd, blk, s);
                return;
            }
        }
        launch_kernel<DIR, BS, BA, false>(c, A, grd, blk, s);
    }

    template <int DIR, int BS, int BA, bool WS>
    static void launch_kernel(hrm_ctx* c, const hrm::SweepArgs& A, dim3 grd, dim3 blk, hipStream_t s)
    {
        // first-order schemes: all double except the float five-equation one
        if ((c->flags & HRM_FOUR_EQ) || ((c->flags & HRM_FIRST_ORDER) && c->precision == HRM_FP64)) {
            hipLaunchKernelGGL((hrm::k_sweep<N, D, DIR, BS, BA, double, 2, WS>), grd, blk, 0, s, A);
            return;
        }
        if constexpr (D <= 2) {
            // learned weights: FP64 face arithmetic, one and two dimensions
            if (c->weights == HRM_WEIGHTS_MLP) {
                hipLaunchKernelGGL((hrm::k_sweep<N, D, DIR, BS, BA, double, 1, WS>), grd, blk, 0, s, A);
                return;
            }
        }
        if (c->precision == HRM_FP32)
            hipLaunchKernelGGL((hrm::k_sweep<N, D, DIR, BS, BA, float, 0, WS>), grd, blk, 0, s, A);
        else
            hipLaunchKernelGGL((hrm::k_sweep<N, D, DIR, BS, BA, double, 0, WS>), grd, blk, 0, s, A);
    }

    // tiles as sweep_tile gives them
    static void sweep(hrm_ctx* c, int dir, hrm::SweepArgs& A, hipStream_t s)
    {
        if constexpr (D == 1) {
            launch_dir<0, 256, 1>(c, A, s);
        } else {
            if (dir == 0) {
                int BS, BA;
                sweep_tile(c, 0, BS, BA);
                if (BA == 1)
                    launch_dir<0, 256, 1>(c, A, s);
                else if (BS == 32)
                    launch_dir<0, 32, 8>(c, A, s);
                else
                    launch_dir<0, 64, 4>(c, A, s);
            }
            if (dir == 1) launch_dir<1, 16, 16>(c, A, s);
            if constexpr (D >= 3)
                if (dir == 2) launch_dir<2, 16, 16>(c, A, s);
        }
    }

    // a stage by k_plane
    static void plane(hrm_ctx* c, const hrm::SweepArgs& S, hipStream_t s)
    {
        if constexpr (D == 2) {
            hrm::PlaneArgs A;
            memset(&A, 0, sizeof(A));
            A.s = S;
            A.s.bclo = c->bclo[0];
            A.s.bchi = c->bchi[0];
            A.s.blo = c->d_bnd[0][0];
            A.s.bhi = c->d_bnd[0][1];
            A.s.idx = 1.0 / c->dx[0];
            A.bclo = c->bclo[1];
            A.bchi = c->bchi[1];
            A.blo = c->d_bnd[1][0];
            A.bhi = c->d_bnd[1][1];
            A.idx = 1.0 / c->dx[1];
            const dim3 grd((c->n[0] + hrm::PLANE_X - 1) / hrm::PLANE_X, (c->n[1] + hrm::PLANE_Y - 1) / hrm::PLANE_Y);
            if (c->precision == HRM_FP32)
                hipLaunchKernelGGL((hrm::k_plane<N, float>), grd, dim3(256), 0, s, A);
            else
                hipLaunchKernelGGL((hrm::k_plane<N, double>), grd, dim3(256), 0, s, A);
        }
    }

    // two cells per thread of a pointwise kernel: planes of nc doubles at 16-byte
    // addresses throughout
    static bool pairs(long long nc, std::initializer_list<const void*> arrays)
    {
        bool ok = nc % 2 == 0;
        for (const void* p : arrays) ok = ok && reinterpret_cast<uintptr_t>(p) % 16 == 0;
        return ok;
    }
    static unsigned cell_blocks(long long nc, int V) { return (unsigned)std::min<long long>((nc + 256 * V - 1) / (256 * V), 8192); }

    static void equilibrium(hrm_ctx* c, const double* W, double* p, double* T, double* cs, hipStream_t s)
    {
        if (pairs(c->ncell, {W, p, T, cs}))
            hipLaunchKernelGGL((hrm::k_equilibrium<N, D, 2>), dim3(cell_blocks(c->ncell, 2)), dim3(256), 0, s, W,
                               c->ncell, c->eos, p, T, cs);
        else
            hipLaunchKernelGGL((hrm::k_equilibrium<N, D, 1>), dim3(cell_blocks(c->ncell, 1)), dim3(256), 0, s, W,
                               c->ncell, c->eos, p, T, cs);
    }

    static void relax(hrm_ctx* c, double* W, hipStream_t s)
    {
        TimerScope t(c, HRM_T_RELAX, s);
        if (pairs(c->ncell, {W}))
            hipLaunchKernelGGL((hrm::k_relax<N, D, 2>), dim3(cell_blocks(c->ncell, 2)), dim3(256), 0, s, W, c->ncell,
                               c->eos, c->d_cnt);
        else
            hipLaunchKernelGGL((hrm::k_relax<N, D, 1>), dim3(cell_blocks(c->ncell, 1)), dim3(256), 0, s, W, c->ncell,
                               c->eos, c->d_cnt);
    }

    // per-block maxima of the cells (ncb blocks), then of the Dirichlet ghost
    // states; returns the number of partial blocks
    static int wavespeed_parts(hrm_ctx* c, const double* W, int ncb, hipStream_t s)
    {
        const int four = (c->flags & HRM_FOUR_EQ) ? 1 : 0;
        if (pairs(c->ncell, {W}))
            hipLaunchKernelGGL((hrm::k_wavespeed<N, D, 2>), dim3(ncb), dim3(256), 0, s, W, c->ncell, c->eos, four, -1,
                               c->d_part);
        else
            hipLaunchKernelGGL((hrm::k_wavespeed<N, D, 1>), dim3(ncb), dim3(256), 0, s, W, c->ncell, c->eos, four, -1,
                               c->d_part);
        int nb = ncb;
        for (int d = 0; d < D; ++d)
            for (int side = 0; side < 2; ++side)
                if (c->d_bnd[d][side]) {
                    hipLaunchKernelGGL((hrm::k_wavespeed<N, D, 1>), dim3(c->nbpart[d]), dim3(256), 0, s,
                                       c->d_bnd[d][side], c->nface[d], c->eos, four, d, c->d_part + (size_t)nb * D);
                    nb += c->nbpart[d];
                }
        return nb;
    }

    // the partials of W in the layout of the final sweep's: nslot slots,
    // then the Dirichlet ghost states
    static void seed_parts(hrm_ctx* c, const double* W, hipStream_t s)
    {
        TimerScope t(c, HRM_T_WAVESPEED, s);
        (void)wavespeed_parts(c, W, c->nslot, s);
    }

    // the time step from the partials of seed_parts or of the last final sweep
    static void reduce_dt(hrm_ctx* c, const hrm::DtArgs& a, double* slot, hipStream_t s)
    {
        TimerScope t(c, HRM_T_WAVESPEED, s);
        int nb = c->nslot;
        for (int d = 0; d < D; ++d)
            for (int side = 0; side < 2; ++side)
                if (c->d_bnd[d][side]) nb += c->nbpart[d];
        hipLaunchKernelGGL((hrm::k_reduce_dt<D>), dim3(1), dim3(hrm::RT), 0, s, c->d_part, nb, c->nslot, c->d_maxs, a,
                           slot);
    }

    static void wavespeed(hrm_ctx* c, const double* W, double* out, hipStream_t s)
    {
        TimerScope t(c, HRM_T_WAVESPEED, s);
        const int nb = wavespeed_parts(c, W, c->npart, s);
        hipLaunchKernelGGL((hrm::k_reduce_max<D>), dim3(1), dim3(hrm::RT), 0, s, c->d_part, nb, out);
    }
};

template <typename Fn>
int dispatch(hrm_ctx* c, Fn&& fn)
{
    switch (c->N * 10 + c->D) {
    case 21: fn(Ops<2, 1>()); return HRM_OK;
    case 22: fn(Ops<2, 2>()); return HRM_OK;
    case 23: fn(Ops<2, 3>()); return HRM_OK;
    case 31: fn(Ops<3, 1>()); return HRM_OK;
    case 32: fn(Ops<3, 2>()); return HRM_OK;
    case 33: fn(Ops<3, 3>()); return HRM_OK;
    default: return fail(c, HRM_EUNSUPPORTED, "N=%s%lld with this dim is not built", "", c->N);
    }
}

hrm::SweepArgs base_args(hrm_ctx* c)
{
    hrm::SweepArgs A;
    memset(&A, 0, sizeof(A));
    A.cnt = c->d_cnt;
    A.ncell = c->ncell;
    for (int d = 0; d < 3; ++d) A.n[d] = c->n[d];
    A.e = c->eos;
    A.P = c->par;
    return A;
}

int check_boundary(hrm_ctx* c);

// The stages that k_plane takes: of 2D grids of up to 2048 tiles (eight a CU,
// 215 000 cells), where it beats the two sweeps (us a step, sweeps / k_plane, two
// species: 127 x 65 62 / 36, 300 x 200 78 / 62, 500 x 300 114 / 94, 700 x 350 144 / 131,
// 1024 x 512 211 / 231; three species: 76 / 43, 93 / 74, 135 / 119, 175 / 169, 255 / 294).
// The limit is eight tiles a CU, between 500 x 300 (1462 tiles: it leads by 13 to
// 21 %) and 700 x 350 (2350 tiles: still 4 to 10 %).  The curves cross above it,
// before 1024 x 512, between sizes that were not timed.  With float faces and three
// species, planes of 16 cells across and over 6000 along are 3 % slower here than
// by the sweeps.
// The first-order schemes, the learned weights and runs with the launch timers on,
// which want the sweeps one by one, are left to the sweeps.
bool plane_fits(const hrm_ctx* c)
{
    const long long tiles =
        ((c->n[0] + hrm::PLANE_X - 1ll) / hrm::PLANE_X) * ((c->n[1] + hrm::PLANE_Y - 1ll) / hrm::PLANE_Y);
    return c->D == 2 && tiles <= 2048 && c->weights == HRM_WEIGHTS_IS &&
           !(c->flags & (HRM_FIRST_ORDER | HRM_FOUR_EQ)) && !c->timing_mask;
}

// all directions of L(W_s); with `stage` the last one applies the stage
// update (and writes the wavespeed partials of its output into wpart)
int run_operator(hrm_ctx* c, const double* Ws, const double* Wn, double* Wout, double* rhs, const double* slot,
                 bool stage, double a, double b, int relax, hipStream_t s, double* wpart = nullptr, int hold = 0,
                 int phase = 0, const hrm::DtArgs* dt = nullptr)
{
    if (c->weights == HRM_WEIGHTS_MLP && !c->mlp_ready)
        return fail(c, HRM_EINVAL, "learned weights selected but hrm_set_mlp not called%s");
    if (const int rb = check_boundary(c)) return rb;
    hrm::SweepArgs A = base_args(c);
    A.Ws = Ws;
    A.Wn = Wn;
    A.Wout = Wout;
    A.rhs = rhs;
    A.slot = slot;
    A.a = a;
    A.b = b;
    A.relax = relax;
    A.hold = hold;
    A.wpart = stage ? wpart : nullptr;
    A.nslot = (unsigned)c->nslot;
    if (phase) {
        A.phase = phase;
        A.part = c->d_part;
        A.npart = c->nslot;
        for (int side = 0; side < 2; ++side)
            if (c->d_bnd[0][side]) A.npart += c->nbpart[0];
        A.tnext = c->d_maxs;
        A.slotw = const_cast<double*>(slot);
        A.dt = *dt;
    }
    int rc = HRM_OK;
    if (stage && plane_fits(c)) {
        rc = dispatch(c, [&](auto ops) { decltype(ops)::plane(c, A, s); });
        return rc != HRM_OK ? rc : check_launch(c, "stage");
    }
    for (int d = 0; d < c->D; ++d) {
        const bool last = d == c->D - 1;
        A.mode = (stage && last) ? hrm::MODE_FINAL : (d == 0 ? hrm::MODE_WRITE : hrm::MODE_ADD);
        rc = dispatch(c, [&](auto ops) { decltype(ops)::sweep(c, d, A, s); });
        if (rc != HRM_OK) return rc;
        if ((rc = check_launch(c, "sweep")) != HRM_OK) return rc;
    }
    return rc;
}

bool valid_ptr(const void* p) { return p != nullptr; }

// every Dirichlet face has had its state set
int check_boundary(hrm_ctx* c)
{
    for (int d = 0; d < c->D; ++d)
        for (int side = 0; side < 2; ++side)
            if (c->d_bnd[d][side] && !c->bnd_set[d][side])
                return fail(c, HRM_EINVAL, "Dirichlet state of dimension %s%lld not set (hrm_set_boundary_state)", "",
                            d);
    return HRM_OK;
}

hrm::DtArgs dt_args(hrm_ctx* c, double cfl, double dt_fixed, double t_end)
{
    hrm::DtArgs a;
    a.D = c->D;
    for (int d = 0; d < 3; ++d) a.dx[d] = c->dx[d];
    a.cfl = cfl;
    a.dt_fixed = dt_fixed;
    a.t_end = t_end;
    return a;
}

// the wavespeed partials of W^n for the first step of a run (the later
// steps find them written by the final sweep of the step before)
int seed_enqueue(hrm_ctx* c, const double* d_W, hipStream_t s)
{
    int rc = check_boundary(c);
    if (rc == HRM_OK) rc = dispatch(c, [&](auto ops) { decltype(ops)::seed_parts(c, d_W, s); });
    if (rc == HRM_OK) rc = check_launch(c, "hrm_advance wavespeed");
    return rc;
}

// the launches of one RK3 step on stream s: time step from the partials,
// three stages with the relaxation, the last one leaving the partials of
// W^{n+1}
int step_enqueue(hrm_ctx* c, double* d_W, double cfl, double dt_fixed, double t_end, double* d_slot, hipStream_t s)
{
    static const double RK_A[3] = {0.0, 3.0 / 4.0, 1.0 / 3.0};
    static const double RK_B[3] = {1.0, 1.0 / 4.0, 2.0 / 3.0};
    const hrm::DtArgs a = dt_args(c, cfl, dt_fixed, t_end);
    int rc = check_boundary(c);
    const bool line = c->D == 1;  // the first sweep takes the time step itself
    if (rc == HRM_OK && !line) rc = dispatch(c, [&](auto ops) { decltype(ops)::reduce_dt(c, a, d_slot, s); });
    if (rc == HRM_OK) rc = check_launch(c, "hrm_advance time step");
    if (rc == HRM_OK)
        rc = run_operator(c, d_W, d_W, c->d_W1, c->d_rhs, d_slot, true, RK_A[0], RK_B[0], 1, s, nullptr, 1,
                          line ? 1 : 0, &a);
    if (rc == HRM_OK)
        rc = run_operator(c, c->d_W1, d_W, c->d_W2, c->d_rhs, d_slot, true, RK_A[1], RK_B[1], 1, s, nullptr, 1,
                          line ? 2 : 0, &a);
    if (rc == HRM_OK)
        rc = run_operator(c, c->d_W2, d_W, d_W, c->d_rhs, d_slot, true, RK_A[2], RK_B[2], 1, s, c->d_part, 1);
    return rc;
}

void drop_graph(hrm_ctx* c)
{
    if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
    c->gexec = nullptr;
}

}  // namespace

extern "C" {

void hrm_default_params(hrm_params* p)
{
    if (!p) return;
    p->eps_weno = 1e-15;
    p->eps_i_ar = 1e-10;
    p->eps_i_a = 1e-10;
    p->hs_i_ar = 1e-11;
    p->hs_i_a = 1e-11;
    p->hs_i_rc2 = 1e-9;
    p->eps_f_ar = 1e-10;
    p->eps_f_a = 1e-10;
    p->eps_f_re = 1e-8;
    p->hs_f_ar = 1e-11;
    p->hs_f_a = 1e-11;
    p->hs_f_re = 1e-9;
    p->Cs = 1e12;
    p->qexp = 2.0;
    p->psi = 256.0 / 175.0;
}

const char* hrm_last_error(const hrm_ctx* ctx) { return ctx ? ctx->err : "NULL context"; }

int hrm_create(const hrm_grid* g, const hrm_eos* e, const hrm_params* prm, hrm_ctx** out)
{
    if (!out) return HRM_EINVAL;
    *out = nullptr;
    if (!g || !e) return HRM_EINVAL;
    if (g->dim < 1 || g->dim > 3) return HRM_EINVAL;
    if (e->nspecies < 2 || e->nspecies > HRM_MAX_SPECIES) return HRM_EINVAL;
    for (int d = 0; d < 3; ++d) {
        if (g->n[d] < 1 || (d >= g->dim && g->n[d] != 1)) return HRM_EINVAL;
        if (d < g->dim && !(g->dx[d] > 0.0)) return HRM_EINVAL;
        if (d < g->dim) {
            for (int side = 0; side < 2; ++side) {
                const int bc = side ? g->bc_hi[d] : g->bc_lo[d];
                if (bc != HRM_BC_TRANSMISSIVE && bc != HRM_BC_PERIODIC && bc != HRM_BC_DIRICHLET) return HRM_EINVAL;
            }
            if ((g->bc_lo[d] == HRM_BC_PERIODIC) != (g->bc_hi[d] == HRM_BC_PERIODIC)) return HRM_EINVAL;
        }
    }
    for (int k = 0; k < e->nspecies; ++k) {
        if (!(e->gamma[k] > 1.0) || !(e->cv[k] > 0.0) || !(e->pinf[k] >= 0.0)) return HRM_EINVAL;
        if (k > 0 && e->pinf[k] != 0.0) return HRM_EINVAL;  // one stiffened gas, species 0 (Sec. 4.2)
    }
    if (g->precision != HRM_FP64 && g->precision != HRM_FP32) return HRM_EINVAL;
    if (g->weights != HRM_WEIGHTS_IS && g->weights != HRM_WEIGHTS_MLP) return HRM_EINVAL;
    if (g->weights == HRM_WEIGHTS_MLP && (g->precision != HRM_FP64 || g->dim > 2)) return HRM_EUNSUPPORTED;

    hrm_ctx* c = new (std::nothrow) hrm_ctx;
    if (!c) return HRM_ENOMEM;
    memset(c, 0, sizeof(*c));
    c->N = e->nspecies;
    c->D = g->dim;
    c->M = 2 * c->N + c->D;
    for (int d = 0; d < 3; ++d) {
        c->n[d] = g->n[d];
        c->dx[d] = d < g->dim ? g->dx[d] : 1.0;
        c->bclo[d] = d < g->dim ? g->bc_lo[d] : HRM_BC_TRANSMISSIVE;
        c->bchi[d] = d < g->dim ? g->bc_hi[d] : HRM_BC_TRANSMISSIVE;
    }
    c->precision = g->precision;
    c->weights = g->weights;
    c->flags = g->flags;
    c->ncell = (long long)g->n[0] * g->n[1] * g->n[2];
    if (!((c->N == 2 || c->N == 3))) {
        delete c;
        return HRM_EUNSUPPORTED;
    }
    if (!sizes_fit(c)) {
        delete c;
        return HRM_EUNSUPPORTED;
    }
    for (int k = 0; k < hrm::MAXN; ++k) {
        const bool on = k < c->N;
        c->eos.g[k] = on ? e->gamma[k] : 2.0;
        c->eos.cv[k] = on ? e->cv[k] : 1.0;
        c->eos.pinf[k] = on ? e->pinf[k] : 0.0;
        c->eos.q[k] = on ? e->q[k] : 0.0;
        c->eos.ig1[k] = 1.0 / (c->eos.g[k] - 1.0);
        c->eos.gpi1[k] = c->eos.g[k] * c->eos.pinf[k] / (c->eos.g[k] - 1.0);
        c->eos.cp[k] = c->eos.g[k] * c->eos.cv[k];
    }
    hrm_params p;
    if (prm)
        p = *prm;
    else
        hrm_default_params(&p);
    hrm::ParDev& P = c->par;
    P.eps_weno = p.eps_weno;
    P.eps_i_ar = p.eps_i_ar;
    P.eps_i_a = p.eps_i_a;
    P.hs_i_ar = p.hs_i_ar;
    P.hs_i_a = p.hs_i_a;
    P.hs_i_rc2 = p.hs_i_rc2;
    P.eps_f_ar = p.eps_f_ar;
    P.eps_f_a = p.eps_f_a;
    P.eps_f_re = p.eps_f_re;
    P.hs_f_ar = p.hs_f_ar;
    P.hs_f_a = p.hs_f_a;
    P.hs_f_re = p.hs_f_re;
    P.Cs = p.Cs;
    P.qexp = p.qexp;
    P.psi = p.psi;
    P.hcs_a = 75.0 * p.psi / 128.0 - 37.0 / 60.0;
    P.hcs_b = 25.0 * p.psi / 256.0 - 2.0 / 15.0;
    P.hcs_c = 3.0 * p.psi / 256.0 - 1.0 / 60.0;
    P.flags = g->flags;
    if (g->flags & HRM_FOUR_EQ) P.flags |= HRM_FIRST_ORDER;  // the direct HRM solver is first order
    P.fast_flux_limiter = p.eps_f_ar >= p.hs_f_ar && p.eps_f_a >= p.hs_f_a && p.eps_f_re >= p.hs_f_re;
    P.fast_interp_limiter = p.eps_i_ar >= p.hs_i_ar && p.eps_i_a >= p.hs_i_a;

    const size_t bytes = sizeof(double) * (size_t)c->M * (size_t)c->ncell;
    c->npart = (int)std::min<long long>((c->ncell + 255) / 256, 2048);
    {
        int BS, BA;
        sweep_tile(c, c->D - 1, BS, BA);
        const dim3 g = sweep_grid(c, c->D - 1, BS, BA);
        // the largest power of two up to the block count and 2048, so that
        // every slot receives at least one block
        const long long nblk = (long long)g.x * g.y * g.z;
        c->nslot = 1;
        while (c->nslot < 2048 && 2ll * c->nslot <= nblk) c->nslot *= 2;
    }
    int nparts = std::max(c->npart, c->nslot);
    if (c->D == 1) nparts = (int)std::max<long long>(nparts, (hrm::line_part(c->ncell) + 2) / 3);
    for (int d = 0; d < 3; ++d) {
        c->nface[d] = c->ncell / c->n[d];
        c->nbpart[d] = (int)std::min<long long>((c->nface[d] + 255) / 256, 256);
        if (d < c->D)
            for (int side = 0; side < 2; ++side)
                if ((side ? c->bchi[d] : c->bclo[d]) == HRM_BC_DIRICHLET) nparts += c->nbpart[d];
    }
    bool ok = true;
    for (int d = 0; d < c->D; ++d)
        for (int side = 0; side < 2; ++side)
            if ((side ? c->bchi[d] : c->bclo[d]) == HRM_BC_DIRICHLET)
                ok = ok && hipMalloc((void**)&c->d_bnd[d][side], sizeof(double) * (size_t)c->M * c->nface[d]) ==
                               hipSuccess;
    if (c->D > 1) ok = ok && hipMalloc((void**)&c->d_rhs, bytes) == hipSuccess;
    ok = ok && hipMalloc((void**)&c->d_W1, bytes) == hipSuccess;
    ok = ok && hipMalloc((void**)&c->d_W2, bytes) == hipSuccess;
    ok = ok && hipMalloc((void**)&c->d_part, sizeof(double) * 3 * (size_t)nparts) == hipSuccess;
    ok = ok && hipMalloc((void**)&c->d_maxs, sizeof(double) * 4) == hipSuccess;
    ok = ok && hipMalloc((void**)&c->d_cnt, sizeof(unsigned long long) * 8) == hipSuccess;
    if (c->weights == HRM_WEIGHTS_MLP) ok = ok && hipMalloc((void**)&c->d_mlp, sizeof(hrm::MlpPacked)) == hipSuccess;
    P.mlp = c->d_mlp;
    if (ok) ok = hipMemset(c->d_cnt, 0, sizeof(unsigned long long) * 8) == hipSuccess;
    if (ok) ok = hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        hrm_destroy(c);
        return HRM_ENOMEM;
    }
    *out = c;
    return HRM_OK;
}

int hrm_destroy(hrm_ctx* c)
{
    if (!c) return HRM_EINVAL;
    (void)hipDeviceSynchronize();
    if (c->pool_ready)
        for (int i = 0; i < 4096; ++i) {
            (void)hipEventDestroy(c->pool[i][0]);
            (void)hipEventDestroy(c->pool[i][1]);
        }
    for (int d = 0; d < 3; ++d)
        for (int side = 0; side < 2; ++side) (void)hipFree(c->d_bnd[d][side]);
    (void)hipFree(c->d_rhs);
    (void)hipFree(c->d_W1);
    (void)hipFree(c->d_W2);
    (void)hipFree(c->d_part);
    (void)hipFree(c->d_maxs);
    (void)hipFree(c->d_cnt);
    (void)hipFree(c->d_mlp);
    drop_graph(c);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    delete c;
    return HRM_OK;
}

int hrm_max_wavespeed(hrm_ctx* c, const double* d_W, double* d_out, void* stream)
{
    if (!c) return HRM_EINVAL;
    if (!valid_ptr(d_W) || !valid_ptr(d_out)) return fail(c, HRM_EINVAL, "hrm_max_wavespeed: NULL pointer%s", "");
    if (const int rb = check_boundary(c)) return rb;
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    const int rc = dispatch(c, [&](auto ops) { decltype(ops)::wavespeed(c, d_W, d_out, s); });
    return rc != HRM_OK ? rc : check_launch(c, "hrm_max_wavespeed");
}

int hrm_compute_dt(hrm_ctx* c, const double* d_maxspeed, double cfl, double dt_fixed, double t_end, double* d_slot,
                   void* stream)
{
    if (!c) return HRM_EINVAL;
    if (!valid_ptr(d_maxspeed) || !valid_ptr(d_slot)) return fail(c, HRM_EINVAL, "hrm_compute_dt: NULL pointer%s");
    if (!(dt_fixed > 0.0) && !(cfl > 0.0)) return fail(c, HRM_EINVAL, "hrm_compute_dt: need cfl > 0 or dt_fixed > 0%s");
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    TimerScope t(c, HRM_T_DT, s);
    hipLaunchKernelGGL(hrm::k_dt, dim3(1), dim3(64), 0, s, d_maxspeed, dt_args(c, cfl, dt_fixed, t_end), d_slot);
    return check_launch(c, "hrm_compute_dt");
}

int hrm_rhs(hrm_ctx* c, const double* d_W, double* d_L, const double* d_slot, void* stream)
{
    if (!c) return HRM_EINVAL;
    if (!valid_ptr(d_W) || !valid_ptr(d_L) || !valid_ptr(d_slot)) return fail(c, HRM_EINVAL, "hrm_rhs: NULL pointer%s");
    if ((const double*)d_L == d_W) return fail(c, HRM_EINVAL, "hrm_rhs: d_L aliases d_W%s");
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    return run_operator(c, d_W, nullptr, nullptr, d_L, d_slot, false, 0.0, 0.0, 0, s);
}

int hrm_rk_stage(hrm_ctx* c, int stage, const double* d_Wn, const double* d_Ws, double* d_Wout, const double* d_slot,
                 void* stream)
{
    static const double RK_A[3] = {0.0, 3.0 / 4.0, 1.0 / 3.0};
    static const double RK_B[3] = {1.0, 1.0 / 4.0, 2.0 / 3.0};
    if (!c) return HRM_EINVAL;
    if (stage < 0 || stage > 2) return fail(c, HRM_EINVAL, "hrm_rk_stage: stage %s%lld not in 0..2", "", stage);
    if (!valid_ptr(d_Wn) || !valid_ptr(d_Ws) || !valid_ptr(d_Wout) || !valid_ptr(d_slot))
        return fail(c, HRM_EINVAL, "hrm_rk_stage: NULL pointer%s");
    if ((const double*)d_Wout == d_Ws) return fail(c, HRM_EINVAL, "hrm_rk_stage: d_Wout aliases d_Ws%s");
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    return run_operator(c, d_Ws, d_Wn, d_Wout, c->d_rhs, d_slot, true, RK_A[stage], RK_B[stage],
                        (c->flags & HRM_FUSE_RELAX) ? 1 : 0, s);
}

int hrm_set_boundary_state(hrm_ctx* c, int dim, int side, const double* d_state, void* stream)
{
    if (!c) return HRM_EINVAL;
    if (dim < 0 || dim >= c->D || side < 0 || side > 1 || !c->d_bnd[dim][side])
        return fail(c, HRM_EINVAL, "hrm_set_boundary_state: face (dim %s%lld) is not a Dirichlet face", "", dim);
    if (!valid_ptr(d_state)) return fail(c, HRM_EINVAL, "hrm_set_boundary_state: NULL pointer%s");
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    if (hipMemcpyAsync(c->d_bnd[dim][side], d_state, sizeof(double) * (size_t)c->M * c->nface[dim],
                       hipMemcpyDeviceToDevice, s) != hipSuccess)
        return fail(c, HRM_EDEVICE, "hrm_set_boundary_state: copy failed: %s", hipGetErrorString(hipGetLastError()));
    c->bnd_set[dim][side] = 1;
    return HRM_OK;
}

int hrm_relax(hrm_ctx* c, double* d_W, void* stream)
{
    if (!c) return HRM_EINVAL;
    if (!valid_ptr(d_W)) return fail(c, HRM_EINVAL, "hrm_relax: NULL pointer%s");
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    const int rc = dispatch(c, [&](auto ops) { decltype(ops)::relax(c, d_W, s); });
    return rc != HRM_OK ? rc : check_launch(c, "hrm_relax");
}

int hrm_equilibrium_state(hrm_ctx* c, const double* d_W, double* d_p, double* d_T, double* d_c, void* stream)
{
    if (!c) return HRM_EINVAL;
    if (!valid_ptr(d_W)) return fail(c, HRM_EINVAL, "hrm_equilibrium_state: NULL state%s");
    if (!d_p && !d_T && !d_c) return HRM_OK;
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    const int rc = dispatch(c, [&](auto ops) { decltype(ops)::equilibrium(c, d_W, d_p, d_T, d_c, s); });
    return rc != HRM_OK ? rc : check_launch(c, "hrm_equilibrium_state");
}

int hrm_set_mlp(hrm_ctx* c, const float* h_params)
{
    if (!c) return HRM_EINVAL;
    if (c->weights != HRM_WEIGHTS_MLP) return fail(c, HRM_EINVAL, "hrm_set_mlp: the grid uses App. C weights%s");
    if (!h_params) return fail(c, HRM_EINVAL, "hrm_set_mlp: NULL parameters%s");
    hrm::MlpPacked pk;
    hrm::mlp_pack_host(h_params, &pk);
    // ordered after the work already enqueued by this context
    if (hipStreamSynchronize(c->last_stream) != hipSuccess ||
        hipMemcpy(c->d_mlp, &pk, sizeof(pk), hipMemcpyHostToDevice) != hipSuccess)
        return fail(c, HRM_EDEVICE, "hrm_set_mlp: copy failed%s");
    c->mlp_ready = 1;
    return HRM_OK;
}

int hrm_mlp_infer(hrm_ctx* c, const double* d_U5, long long n, double* d_val, float* d_omega, void* stream)
{
    if (!c) return HRM_EINVAL;
    if (c->weights != HRM_WEIGHTS_MLP || !c->mlp_ready)
        return fail(c, HRM_EINVAL, "hrm_mlp_infer: no learned weights on this grid%s");
    if (n < 0 || (n > 0 && (!valid_ptr(d_U5) || !valid_ptr(d_val) || !d_omega)))
        return fail(c, HRM_EINVAL, "hrm_mlp_infer: bad arguments%s");
    if (n == 0) return HRM_OK;
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    hipLaunchKernelGGL(hrm::k_mlp_infer, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, c->d_mlp, d_U5, n,
                       c->par.eps_weno, d_val, d_omega);
    return check_launch(c, "hrm_mlp_infer");
}

int hrm_advance(hrm_ctx* c, double* d_W, int nsteps, double cfl, double dt_fixed, double t_end, double* d_slot,
                void* stream)
{
    if (!c) return HRM_EINVAL;
    if (!valid_ptr(d_W) || !valid_ptr(d_slot)) return fail(c, HRM_EINVAL, "hrm_advance: NULL pointer%s");
    if (nsteps < 0) return fail(c, HRM_EINVAL, "hrm_advance: nsteps = %s%lld < 0", "", nsteps);
    if (!(dt_fixed > 0.0) && !(cfl > 0.0)) return fail(c, HRM_EINVAL, "hrm_advance: need cfl > 0 or dt_fixed > 0%s");
    if (c->weights == HRM_WEIGHTS_MLP && !c->mlp_ready)
        return fail(c, HRM_EINVAL, "learned weights selected but hrm_set_mlp not called%s");
    if (nsteps == 0) return HRM_OK;
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    // a line: one step in a launch, or up to LINE_STEPS where one workgroup holds it
    // (the launch timers want the sweeps one by one)
    if (c->D == 1 && !c->timing_mask && hrm::line_fits(c->n[0], c->par.flags, c->precision, c->weights)) {
        if (const int rb = check_boundary(c)) return rb;
        hrm::LineArgs A;
        memset(&A, 0, sizeof(A));
        A.W = d_W;
        A.slot = d_slot;
        A.cnt = c->d_cnt;
        A.n = c->n[0];
        A.nsteps = nsteps;
        A.bclo = c->bclo[0];
        A.bchi = c->bchi[0];
        A.blo = c->d_bnd[0][0];
        A.bhi = c->d_bnd[0][1];
        A.idx = 1.0 / c->dx[0];
        A.dt = dt_args(c, cfl, dt_fixed, t_end);
        A.e = c->eos;
        A.P = c->par;
        if (c->n[0] <= hrm::line_cells(c->N, c->par.flags, c->precision))
            hrm::line_launch(c->N, c->precision, A, s);
        else
            hrm::line_steps(c->N, c->precision, A, c->d_W1, c->d_part, s);
        return check_launch(c, "hrm_advance line");
    }
    int rc = seed_enqueue(c, d_W, s);
    if (rc != HRM_OK) return rc;
    if ((c->flags & HRM_NO_GRAPH) || c->timing_mask) {
        for (int k = 0; k < nsteps && rc == HRM_OK; ++k) rc = step_enqueue(c, d_W, cfl, dt_fixed, t_end, d_slot, s);
        return rc;
    }
    const bool same = c->gexec && c->g_W == d_W && c->g_slot == d_slot && c->g_cfl == cfl &&
                      c->g_dt_fixed == dt_fixed && c->g_t_end == t_end;
    if (!same) {
        drop_graph(c);
        if (hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed) != hipSuccess)
            return fail(c, HRM_EDEVICE, "hrm_advance: stream capture failed%s");
        rc = step_enqueue(c, d_W, cfl, dt_fixed, t_end, d_slot, c->cap_stream);
        hipGraph_t g = nullptr;
        const hipError_t ec = hipStreamEndCapture(c->cap_stream, &g);
        if (rc != HRM_OK || ec != hipSuccess || !g) {
            if (g) (void)hipGraphDestroy(g);
            return rc != HRM_OK ? rc : fail(c, HRM_EDEVICE, "hrm_advance: end capture: %s", hipGetErrorString(ec));
        }
        const hipError_t ei = hipGraphInstantiate(&c->gexec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (ei != hipSuccess) {
            c->gexec = nullptr;
            return fail(c, HRM_EDEVICE, "hrm_advance: graph instantiate: %s", hipGetErrorString(ei));
        }
        c->g_W = d_W;
        c->g_slot = d_slot;
        c->g_cfl = cfl;
        c->g_dt_fixed = dt_fixed;
        c->g_t_end = t_end;
    }
    for (int k = 0; k < nsteps; ++k)
        if (hipGraphLaunch(c->gexec, s) != hipSuccess)
            return fail(c, HRM_EDEVICE, "hrm_advance: graph launch: %s", hipGetErrorString(hipGetLastError()));
    return HRM_OK;
}

int hrm_step(hrm_ctx* c, double* d_W, double cfl, double dt_fixed, double t_end, double* d_slot, void* stream)
{
    return hrm_advance(c, d_W, 1, cfl, dt_fixed, t_end, d_slot, stream);
}

int hrm_get_diagnostics(hrm_ctx* c, hrm_diag* out)
{
    if (!c || !out) return HRM_EINVAL;
    if (hipStreamSynchronize(c->last_stream) != hipSuccess ||
        hipMemcpy(out, c->d_cnt, sizeof(hrm_diag), hipMemcpyDeviceToHost) != hipSuccess) {
        snprintf(c->err, sizeof(c->err), "hrm_get_diagnostics: %s", hipGetErrorString(hipGetLastError()));
        return HRM_EDEVICE;
    }
    return out->relax_bad ? HRM_EADMISSIBLE : HRM_OK;
}

int hrm_reset_diagnostics(hrm_ctx* c, void* stream)
{
    if (!c) return HRM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    c->last_stream = s;
    hipLaunchKernelGGL(hrm::k_zero_u64, dim3(1), dim3(64), 0, s, c->d_cnt, 8);
    return check_launch(c, "hrm_reset_diagnostics");
}

int hrm_set_timing(hrm_ctx* c, int mask)
{
    if (!c) return HRM_EINVAL;
    if (mask && !c->pool_ready) {
        for (int i = 0; i < 4096; ++i)
            if (hipEventCreate(&c->pool[i][0]) != hipSuccess || hipEventCreate(&c->pool[i][1]) != hipSuccess) {
                snprintf(c->err, sizeof(c->err), "hrm_set_timing: %s", hipGetErrorString(hipGetLastError()));
                return HRM_EDEVICE;
            }
        c->pool_ready = 1;
    }
    c->timing_mask = mask;
    return HRM_OK;
}

int hrm_get_timing(hrm_ctx* c, double* ms, long long* counts)
{
    if (!c || !ms || !counts) return HRM_EINVAL;
    if (hipStreamSynchronize(c->last_stream) != hipSuccess) {
        snprintf(c->err, sizeof(c->err), "hrm_get_timing: %s", hipGetErrorString(hipGetLastError()));
        return HRM_EDEVICE;
    }
    fold_timers(c);
    for (int k = 0; k < HRM_NTIMERS; ++k) {
        ms[k] = c->tms[k];
        counts[k] = c->tcnt[k];
        c->tms[k] = 0.0;
        c->tcnt[k] = 0;
    }
    return HRM_OK;
}

}  // extern "C"
