"""Edges of the device arithmetic that no grid reaches by itself, on the CPU:
hrm_device.hpp compiled for the host, the hardware's reciprocal and root
replaced by the host's rounded to 26 bits (about what v_rcp_f64 gives).
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>
using std::isfinite;
#define __device__
#define __forceinline__ inline
#define asm
#define volatile(...)
struct dim3_ { unsigned x, y, z; };
static dim3_ threadIdx, blockDim;
static inline double crude(double x)
{
    uint64_t u;
    memcpy(&u, &x, 8);
    if (std::isfinite(x)) u &= ~((uint64_t(1) << 27) - 1);
    memcpy(&x, &u, 8);
    return x;
}
#define __builtin_amdgcn_rcp(x) crude(1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsq(x) crude(1.0 / std::sqrt(x))
#define __builtin_amdgcn_class(x, mask) ((x) == 0.0 || (x) == INFINITY)
#define __builtin_amdgcn_kernarg_segment_ptr() 0
#define __builtin_amdgcn_ds_bpermute(i, v) (v)
static inline int __lane_id() { return 0; }
static inline unsigned long long __ballot(bool b) { return b; }
static inline double __shfl_xor(double v, int, int) { return v; }
static inline void __syncthreads() {}
template <typename T> static inline void atomicAdd(T* p, T v) { *p += v; }
"""

MAIN = r"""
#include <cstdio>
#include "hrm_device.hpp"
using namespace hrm;

static EosDev eos()
{
    // a stiffened liquid and a gas
    EosDev e;
    memset(&e, 0, sizeof e);
    const double g[2] = {4.4, 1.4}, cp[2] = {4200.0, 1007.0}, pinf[2] = {6e8, 0.0};
    for (int k = 0; k < 2; ++k) {
        e.g[k] = g[k], e.cp[k] = cp[k], e.cv[k] = cp[k] / g[k], e.pinf[k] = pinf[k];
        e.ig1[k] = 1.0 / (g[k] - 1.0), e.gpi1[k] = g[k] * pinf[k] / (g[k] - 1.0);
    }
    return e;
}

// gas that leaves a face on both sides faster than the half cells hold it
static bool emptied(double bound, double loss, double energy)
{
    EosDev e = eos();
    ParDev P;
    memset(&P, 0, sizeof P);
    P.eps_f_ar = P.eps_f_a = bound;
    P.eps_f_re = 1e-8;
    P.fast_flux_limiter = 1;
    St<2, 1> L, R;
    memset(&L, 0, sizeof L);
    L.ar[1] = L.rho = 1.0, L.al[1] = 1.0, L.p = 1e5, L.E = 2.5e5;
    R = L;
    // W+ = W - 2 lam (G - F), W- = W + 2 lam (G - F): one side at a time
    double G[5] = {0.0, loss, 1e5, energy, 0.0}, Gp[1] = {0.0};
    return flux_limit_clean<2, 1, 0>((KArg)&e, (KArg)&P, L, R, 0.5, G, Gp);
}

int main()
{
    printf("%d%d%d%d\n", sqrt_rn(0.0) == 0.0, sqrt_rn(INFINITY) == INFINITY, std::isnan(sqrt_rn(-1.0)), std::isnan(sqrt_rn(NAN)));
    // a gas at p = 0: rho c^2 = 0, so c = 0
    St<2, 1> s;
    memset(&s, 0, sizeof s);
    s.ar[1] = 1.0, s.al[0] = 0.0, s.u[0] = 3.0;
    complete_from_prim<2, 1, double>(eos(), s);
    printf("%d%d\n", s.rc2 == 0.0, s.c == 0.0);
    St<2, 1, float> f;
    memset(&f, 0, sizeof f);
    f.ar[1] = 1.0f, f.al[0] = 0.0;
    complete_from_prim<2, 1, float>(eos(), f);
    printf("%d\n", f.c == 0.0f);
    const double W[5] = {0.0, 1.0, 0.0, 0.0, 0.0};
    state_from_W<2, 1>(eos(), W, s);
    printf("%d\n", s.c == 0.0);
    // a volume fraction below its bound; half-cell densities of both signs under
    // bounds that admit them; an undisturbed face under these
    printf("%d%d%d%d\n", emptied(1e-10, 0.0, 0.0), emptied(-1e30, 3.0, 1e7), emptied(-1e30, -3.0, -1e7),
           emptied(-1e30, 0.0, 0.0));
    int wrong = 0;
    unsigned long long r = 88172645463325252ull;
    for (int i = 0; i < 2000000; ++i) {
        double v[2];
        for (double& x : v) {
            r ^= r << 13, r ^= r >> 7, r ^= r << 17;
            x = std::ldexp(1.0 + (double)(r >> 11) * 0x1p-53, (int)(r % 80) - 40);
        }
        wrong += div_rn(v[0], v[1]) != v[0] / v[1];
        wrong += sqrt_rn(v[0]) != std::sqrt(v[0]);
    }
    printf("%d\n", wrong);
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("edges")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "edges")
    subprocess.run(["g++", "-O2", "-mfma", "-std=c++17", "-ffp-contract=off", "-w", "-I", str(d), "-I",
                    os.path.join(ROOT, "paper_2208_04488_amd", "csrc"), str(d / "main.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()


def test_roots_of_zero_and_infinity(lines):
    assert lines[0] == "1111"


def test_sound_speed_of_a_gas_without_pressure(lines):
    assert lines[1:4] == ["11", "1", "1"]


def test_half_cells_without_density_go_to_the_limiter(lines):
    """A bound that admits them does not make their energy check pass."""
    assert lines[4] == "0001"


def test_quotients_and_roots_round_as_ieee(lines):
    assert lines[5] == "0"
