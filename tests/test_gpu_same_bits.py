"""The kernels of short lines (k_line), longer lines (k_line_step) and small
planes (k_plane) against the sweeps, which the launch timers select: the same
arithmetic in one written order, so the state, the time step and every count
agree to the bit.
"""
import numpy as np
import pytest

from paper_2208_04488_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2208_04488_amd import hrm
    return hrm


def _same(H, prob, steps, flags=0, precision=None):
    import torch
    runs = []
    for sweeps in (False, True):
        s = H.Solver(prob, flags=H.FUSE_RELAX | flags, precision=H.FP64 if precision is None else precision)
        if sweeps:
            H.hrm_set_timing(s.ctx, 1)
        s.advance(steps, cfl=0.4)
        torch.cuda.synchronize()
        runs.append((s.W.clone(), s.slot.clone(), s.diagnostics()))
        s.close()
    (a, sa, da), (b, sb, db) = runs
    assert torch.isfinite(b).all()
    assert torch.equal(a, b), "%d values differ" % int((a != b).sum())
    assert torch.equal(sa, sb)
    assert da == db


# the block sizes of k_line, its last line and the first of k_line_step (447 and
# 383 cells, 511 at first order), whole tiles of k_line_step and one cell more
@pytest.mark.parametrize("n", [1, 2, 3, 64, 255, 256, 383, 384, 447, 448, 511, 512, 711, 712, 1246, 5000])
@pytest.mark.parametrize("kind", ["open", "periodic", "dirichlet", "three", "fp32", "three_fp32", "first", "four_eq"])
def test_lines(H, n, kind):
    base = I.shock_interface(n) if kind.startswith("three") else I.config1(n)
    bc = {"periodic": (I.PERIODIC, I.PERIODIC), "dirichlet": (I.DIRICHLET, I.TRANSMISSIVE)}.get(kind, (0, 0))
    prob = I.Problem(base.name, base.eos, 1, base.n, base.dx, [bc], base.W, cfl=0.4)
    if kind == "dirichlet":
        prob.boundary = {(0, 0): np.ascontiguousarray(base.W[:, 0, 0, :1])}
    flags = {"first": H.FIRST_ORDER, "four_eq": H.FOUR_EQ}.get(kind, 0)
    _same(H, prob, 5, flags, H.FP32 if kind.endswith("fp32") else H.FP64)


def test_longest_line_without_the_sweeps(H):
    _same(H, I.config1(307200), 1)


# whole tiles of 15 x 7, one cell more and one less, grids narrower than a stencil,
# the largest number of tiles
@pytest.mark.parametrize("n", [(1, 1), (2, 9), (14, 6), (15, 7), (16, 8), (30, 14), (127, 65), (480, 448)])
@pytest.mark.parametrize("kind", ["open", "periodic", "inflow", "three", "fp32", "three_fp32"])
def test_planes(H, n, kind):
    """Liquid drops in gas with a jump of the pressure, so that the limiters act."""
    three = kind.startswith("three")
    eos = I.eos_of(I.LIQ_B, I.AIR, I.HELIUM) if three else I.eos_of(I.LIQ_A, I.AIR)
    x, y = np.meshgrid((np.arange(n[0]) + 0.5) / n[0], (np.arange(n[1]) + 0.5) / n[1])
    wave = 0.5 * (np.cos(4 * np.pi * x) + np.cos(4 * np.pi * y + 1))
    liq = I.TRACE + (1 - 4 * I.TRACE) * 0.5 * (1 + np.tanh((wave - 0.3) * 40))
    alpha = [liq, 0.3 * (1 - liq), 0.7 * (1 - liq)] if three else [liq, 1 - liq]
    u = [200.0 * np.sin(2 * np.pi * x), 150.0 * np.sin(2 * np.pi * y + 1)]
    W = I.equilibrium_state(eos, alpha, u, 1e5 * (1 + 0.2 * wave + 9.0 * (x < 0.3)), 300.0 + 20 * wave)
    W = np.ascontiguousarray(W.reshape((W.shape[0], 1, n[1], n[0])))
    bc = {"periodic": [(I.PERIODIC,) * 2] * 2, "inflow": [(I.DIRICHLET, 0), (0, I.DIRICHLET)]}.get(kind, [(0, 0)] * 2)
    prob = I.Problem("plane", eos, 2, n, (1.0 / max(n),) * 2, bc, W)
    if kind == "inflow":
        prob.boundary = {(0, 0): np.ascontiguousarray(W[:, :, :, 0]), (1, 1): np.ascontiguousarray(W[:, :, -1, :])}
    _same(H, prob, 5, precision=H.FP32 if kind.endswith("fp32") else H.FP64)


def _line(kind, n):
    if kind == "three":
        return I.shock_interface(n)
    if kind == "four_eq":
        return I.shock_tube(n)
    return I.config1(n)


# lines beyond one workgroup, whose maximum wavespeed comes from a pass of its own
# before the first step and from the step before in every other; learned weights
# and the timers take the sweeps, the first of which forms the time step
@pytest.mark.parametrize("steps", [4, 5])
@pytest.mark.parametrize("kind", ["plain", "three", "fp32", "dirichlet", "first", "four_eq", "four_eq_dirichlet",
                                  "learned", "learned_dirichlet", "timers_dirichlet", "timers_four_eq"])
def test_steps_of_a_long_line(H, kind, steps):
    """hrm_advance(K) against K calls of hrm_step."""
    import torch
    from paper_2208_04488_amd import learned
    base = _line("four_eq" if "four_eq" in kind else kind, 1003)
    bc = (I.DIRICHLET, I.TRANSMISSIVE) if kind.endswith("dirichlet") else (0, 0)
    prob = I.Problem(base.name, base.eos, 1, base.n, base.dx, [bc], base.W, cfl=0.4)
    if kind.endswith("dirichlet"):
        # faster than any cell: the ghost state sets the time step
        ghost = base.W[:, 0, 0, :1].copy()
        ghost[base.eos.N] += 3000.0 * ghost[:base.eos.N].sum()
        ghost[base.eos.N + 1] += 0.5 * 3000.0 ** 2 * ghost[:base.eos.N].sum()
        prob.boundary = {(0, 0): np.ascontiguousarray(ghost)}
    flags = H.FUSE_RELAX | (H.FIRST_ORDER if kind == "first" else H.FOUR_EQ if "four_eq" in kind else 0)
    p = learned.init_params(5, last_scale=0.3) if kind.startswith("learned") else None
    runs = []
    for whole in (True, False):
        s = H.Solver(prob, flags=flags, precision=H.FP32 if kind == "fp32" else H.FP64, mlp=p)
        if kind.startswith("timers"):
            H.hrm_set_timing(s.ctx, 1)
        for _ in range(1 if whole else steps):
            s.advance(steps, cfl=0.4) if whole else s.step(cfl=0.4)
        torch.cuda.synchronize()
        runs.append((s.W.clone(), s.slot.clone(), s.diagnostics()))
        s.close()
    (a, sa, da), (b, sb, db) = runs
    assert torch.isfinite(a).all() and float(sa[0]) > 0.0
    assert torch.equal(a, b) and torch.equal(sa, sb) and da == db


@pytest.mark.parametrize("species", [2, 3])
@pytest.mark.parametrize("D", [1, 2, 3])
def test_sound_speed_of_the_relaxed_model(H, species, D):
    """The four-equation model's c of hrm_equilibrium_state and of the wavespeed pass, one cell at rest at a time."""
    import torch
    eos = I.eos_of(I.LIQ_B, I.AIR, I.HELIUM) if species == 3 else I.eos_of(I.LIQ_A, I.AIR)
    W = I.random_admissible(eos, D, 64, seed=11, p_range=(1e4, 1e8), u_scale=100.0)
    M = W.shape[0]
    mom = W[species:species + D]
    W[species + D] -= 0.5 * (mom ** 2).sum(axis=0) / W[:species].sum(axis=0)
    mom[...] = 0.0
    one = np.ascontiguousarray(W[:, :1].reshape((M, 1, 1, 1)))
    prob = I.Problem("cell", eos, D, (1,) * D, (1.0,) * D, [(0, 0)] * D, one)
    s = H.Solver(prob, flags=H.FUSE_RELAX | H.FOUR_EQ)
    for i in range(W.shape[1]):
        s.set_state(np.ascontiguousarray(W[:, i].reshape((M, 1, 1, 1))))
        c = s.equilibrium()[2].ravel()[0]
        assert np.isfinite(c) and (s.wavespeed() == c).all(), i
    s.close()
