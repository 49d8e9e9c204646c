"""Bits of runs with learned weights.  The network's inputs are rounded to
bfloat16, so another last bit of a characteristic field is now and then another
input and another weight, which ten steps carry to 1e-6 to 7e-5 of the momentum
beside it.  The order of operations of these runs is therefore fixed, and their
results are kept: tests/golden/learned_weights.npz holds the initial states, the
networks and the states after ten steps of two planes and a line that are
sensitive to it, as the library gave them at commit 347c2d5.
"""
import os

import numpy as np
import pytest

from paper_2208_04488_amd import inputs as I

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "learned_weights.npz")


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2208_04488_amd import hrm
    return hrm


@pytest.mark.parametrize("name", ["plane_3_40x14", "plane_3_36x16", "line_3_150"])
def test_learned_runs_keep_their_bits(H, name):
    import torch
    with np.load(GOLDEN) as z:
        W, out, slot, net = (z[name + k] for k in ("_in", "_out", "_slot", "_net"))
    D, N = (2 if name.startswith("plane") else 1), 3
    n = (W.shape[3], W.shape[2])[:D]
    b = [(H.BC_TRANSMISSIVE, H.BC_TRANSMISSIVE), (H.BC_PERIODIC, H.BC_PERIODIC)][:D]
    e = I.eos_of(I.LIQ_B, I.AIR, I.HELIUM)
    s = H.Solver(I.Problem(name, e, D, n, (1.0 / n[0],) * D, b, W), mlp=net)
    s.advance(10, cfl=0.4)
    torch.cuda.synchronize()
    got, clock = s.state().reshape(W.shape), s.slot[:5].cpu().numpy()
    s.close()
    u, v = got[N:N + D], out[N:N + D]
    print(name, "momentum off by %.1e of its rms" % (np.abs(u - v).max() / np.sqrt((v * v).mean())))
    assert np.array_equal(got, out)
    assert np.array_equal(clock, slot)
