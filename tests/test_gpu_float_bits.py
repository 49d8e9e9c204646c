"""Bits of runs with float faces.  A float face rounds doubles to float (the
node differences, the blending weight, the interpolated state), so another last
bit of one of those doubles, of the time step or of a limiter's theta is now
and then another float, which ten steps carry to 1e-7 to 6e-6 of the momentum
beside it.  The order of operations of these runs is therefore fixed, and their
results are kept: tests/golden/float_faces.npz holds initial states and the
states after ten steps of four shock tubes and one plane that are sensitive to
it, as the library gave them at commit 347c2d5.
"""
import os

import numpy as np
import pytest

from paper_2208_04488_amd import inputs as I

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "float_faces.npz")
TUBES = ["tube_3_46", "tube_3_71", "tube_3_169", "tube_2_382"]


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2208_04488_amd import hrm
    return hrm


def _eos(name):
    return I.eos_of(I.LIQ_B, I.AIR, I.HELIUM) if "_3_" in name else I.eos_of(I.LIQ_A, I.AIR)


def _deviation(got, ref, N, D):
    u, v = got[N:N + D], ref[N:N + D]
    return np.abs(u - v).max() / np.sqrt((v * v).mean())


@pytest.mark.parametrize("shape", [None, (256, 512, 10), (64, 3, 5)])
def test_ensembles_keep_their_bits(H, shape):
    """The tubes in one ensemble per species count, at the default launch shape and at two others."""
    import torch
    with np.load(GOLDEN) as z:
        gold = {k: z[k] for k in z.files}
    for N in (3, 2):
        names = [t for t in TUBES if f"_{N}_" in t]
        W = np.ascontiguousarray(np.concatenate([gold[t + "_in"] for t in names], axis=1))
        n = [gold[t + "_in"].shape[1] for t in names]
        off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
        e = _eos(names[0])
        b = H.hrm_batch_create(H.make_eos(e.gamma, e.cv, e.pinf, e.q), None, off, 1.0 / np.array(n), H.FP32)
        if shape:
            H.hrm_batch_configure(b, *shape)
        d = torch.from_numpy(W).cuda()
        H.hrm_batch_run(b, d, 10, 0.4)
        torch.cuda.synchronize()
        H.hrm_batch_destroy(b)
        got = d.cpu().numpy()
        for t, a in zip(names, off):
            out = gold[t + "_out"]
            mine = got[:, a:a + out.shape[1]]
            print(t, "momentum off by %.1e of its rms" % _deviation(mine, out, N, 1))
            assert np.array_equal(mine, out), t


@pytest.mark.parametrize("name", TUBES + ["plane_3_24x20"])
@pytest.mark.parametrize("sweeps", [False, True])
def test_grids_keep_their_bits(H, name, sweeps):
    """The same states as grids: lines and a plane, by their own kernels and (launch timers on) by the sweeps."""
    import torch
    with np.load(GOLDEN) as z:
        W, out, slot = z[name + "_in"], z[name + "_out"], z[name + "_slot"] if name + "_slot" in z.files else None
    N, D = int(name.split("_")[1]), 2 if name.startswith("plane") else 1
    W = np.ascontiguousarray(W.reshape(W.shape[0], 1, -1, W.shape[-1]))
    n = W.shape[3:] if D == 1 else (W.shape[3], W.shape[2])
    s = H.Solver(I.Problem(name, _eos(name), D, tuple(n), (1.0 / n[0],) * D, [(0, 0)] * D, W), precision=H.FP32)
    if sweeps:
        H.hrm_set_timing(s.ctx, 1)
    s.advance(10, cfl=0.4)
    torch.cuda.synchronize()
    got = s.state().reshape(W.shape[0], -1)
    out = out.reshape(W.shape[0], -1)
    print(name, "momentum off by %.1e of its rms" % _deviation(got, out, N, D))
    assert np.array_equal(got, out)
    if slot is not None:
        assert np.array_equal(s.slot[:5].cpu().numpy(), slot)
    s.close()
