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
