"""FBP where the products of distance and sampling are so large (3.2e5 samples) that FP32 distances
do not prove the staged windows: the kernel with the clamped index, one transducer a chunk. FP32
cannot place such a sample to better than a tenth of one, so the data are constant in time, where
the place matters only through its floor, which is decided exactly; against the FP64 oracle at the
gates of the other FBP tests."""
import math

import numpy as np
import pytest

from checks import BF16_ELEM, check
from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_fine_sampling_of_far_transducers(dtype):
    import torch
    from paper_1304_2017_amd.oat import Plan
    q, dx, rs, c0, n = 24, 1.8, 3240.0, 1.5, 12
    dt = dx / (c0 * 180.0)
    sigma, t0 = dx / (c0 * dt), (rs - 1.28) / c0
    xyz = synth.fibonacci_sphere(q, rs)
    assert 16 * 2.0 ** -24 * (np.abs(xyz).max() / dx * sigma + t0 / dt) > 0.5
    geom = synth.Geometry(n, n, n, dx, synth.centred_origin(n, dx), synth.centred_origin(n, dx),
                          synth.centred_origin(n, dx), xyz, 256, dt, t0, c0, 1.0,
                          np.full(q, 4 * math.pi * rs * rs / q))
    amp = np.random.default_rng(3).normal(size=(q, 1))
    p = torch.from_numpy(np.repeat(amp, geom.n_t, axis=1).astype(np.float32)).to(
        getattr(torch, dtype)).cuda()
    plan = Plan(geom, 0)
    f = plan.fbp(p, out_dtype=p.dtype)
    want = ref.fbp(geom.as_dict(), p.double().cpu().numpy())
    got = f.double().cpu().numpy()
    gates = (1e-5,) if dtype == "float32" else (2e-3, BF16_ELEM)
    check(f"far FBP {dtype}", got, want, *gates)
    flat = np.abs(want) < 10 * np.median(np.abs(want))      # no record begins or ends there
    assert flat.mean() > 0.9
    check(f"far FBP {dtype}, away from the records' ends", got[flat], want[flat], *gates)
    plan.close()
