"""FBP where a tile spans thousands of samples (a node spacing of up to 366 samples, records of up to
256 samples): the staged windows of 4097 to 8192 samples.  The data are constant in time, where a
sample's place matters through its floor alone, which is decided exactly: the FP32 gate of the other
FBP tests, and BF16 images are the FP32 ones rounded once.  Wider windows are refused."""
import math

import numpy as np
import pytest

from checks import check
from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


def _geometry(sigma, n=12, q=20, dx=1.8, rs=108.0, c0=1.5):
    dt = dx / (c0 * sigma)
    o = synth.centred_origin(n, dx)
    return synth.Geometry(n, n, n, dx, o, o, o, synth.fibonacci_sphere(q, rs), 256, dt, (rs - 1.28) / c0, c0,
                          1.0, np.full(q, 4 * math.pi * rs * rs / q))


@pytest.mark.parametrize("sigma", [180.0, 184.0, 300.0, 366.0])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_wide_windows(sigma, dtype):
    import torch
    from paper_1304_2017_amd.oat import Plan
    geom = _geometry(sigma)
    amp = np.random.default_rng(3).normal(size=(geom.n_det, 1))
    p = torch.from_numpy(np.repeat(amp, geom.n_t, axis=1).astype(np.float32)).to(
        getattr(torch, dtype)).cuda()
    plan = Plan(geom, 0)
    f, fb = plan.fbp(p, out_dtype=torch.float32), plan.fbp(p, out_dtype=torch.bfloat16)
    plan.close()
    want = ref.fbp(geom.as_dict(), p.double().cpu().numpy())
    assert np.abs(want).max() > 0
    check(f"FBP {sigma:g} {dtype}", f.double().cpu().numpy(), want, 1e-5)
    assert torch.equal(fb, f.bfloat16())


def test_wider_windows_are_refused():
    import torch
    from paper_1304_2017_amd import oat
    geom = _geometry(368.0)
    plan = oat.Plan(geom, 0)
    with pytest.raises(oat.OatError):
        plan.fbp(torch.zeros((geom.n_det, geom.n_t), device="cuda"))
    plan.close()
