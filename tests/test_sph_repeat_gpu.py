"""H_sph gives the same bits on every call, also where the voxels are taken in several parts (128
transducers or fewer) whose FP64 sums are added.

The outputs are rounded to FP32, which hides differences of 1e-15 between FP64 sums.  So the grid is
symmetric and the image antisymmetric about the plane x = 0 that holds every transducer: the exact
result is zero, what is returned is the rounding of the FP64 sums itself, and any other split of the
voxels, or order of the sums, shows in it."""
import numpy as np
import pytest
import torch

from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,faces", [(5, 0), (16, 0), (100, 0), (128, 0), (20, 2)])
def test_repeated_projections_are_equal(q, faces):
    from paper_1304_2017_amd.oat import Plan
    n, dx, rs, n_f, df = 48, 0.5, 40.0, 64, 0.05
    a = 2.0 * np.pi * (np.arange(q) + 0.3) / q
    xyz = rs * np.stack([np.zeros(q), np.cos(a), np.sin(a)], 1)
    o = synth.centred_origin(n, dx)
    plan = Plan(synth.Geometry(n, n, n, dx, o, o, o, xyz, 256, 0.1, 0.0, 1.5, 1.0), 0,
                arc_table=False, segment_table=False)
    if faces:
        plan.set_aperture(1.0, 1.0, faces)
    g = torch.Generator().manual_seed(q)
    x = torch.randn((n, n, n), generator=g)
    size = plan.sph_project(x.cuda(), n_f, df, df).abs().max()
    x = (x - x.flip(2)).cuda()
    u = plan.sph_project(x, n_f, df, df)
    # a face's nodes have distances that agree to rounding only; a centre's agree exactly
    assert float(u.abs().max()) < 1e-12 * float(size)
    for k in range(40):
        assert torch.equal(plan.sph_project(x, n_f, df, df), u), f"call {k} differs"
    plan.close()
