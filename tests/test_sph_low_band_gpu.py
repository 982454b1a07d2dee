"""H_sph of one short run of frequencies from 0 (or from where every phase is a fraction of a turn),
and a few more: the plain sums over such a band are exact to their outputs' rounding to FP32, and so has the interval
path to be.  The error against FP64 may exceed that of the exact values rounded once by no more than
5e-9 of the 2-norm (eight moments an interval: about 1e-9; six: 2e-8) in quadrature."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_f,f_min,df,faces", [(16, 0.0, 0.3125, 0), (32, 0.0, 0.15625, 0), (7, 0.0, 0.1, 0),
                                                (36, 0.0, 0.139, 0),
                                                (16, 0.002, 0.05, 0), (20, 0.0, 0.2, 2), (1, 0.01, 0.5, 0)])
@pytest.mark.parametrize("image", ["iterate", "phantom", "smooth"])
def test_as_exact_as_the_plain_sums(n_f, f_min, df, faces, image):
    from paper_1304_2017_amd.oat import Plan
    shape, q, dx = (33, 37, 40), 200, 0.4
    o = [synth.centred_origin(n, dx) for n in reversed(shape)]
    geom = synth.Geometry(*reversed(shape), dx, *o, synth.fibonacci_sphere(q, 40.0), 256, 0.05, 0.0, 1.5, 1.0)
    plan = Plan(geom, 0, arc_table=False, segment_table=False)
    ap = (2.0, 1.5, faces) if faces else None
    if faces:
        plan.set_aperture(*ap)
    rng = np.random.default_rng(n_f)
    x = rng.normal(size=shape)
    if image == "phantom":
        x *= rng.random(shape) < 0.05
    elif image == "smooth":
        x = 1.0 + 0.1 * x
    x = torch.from_numpy(x.astype(np.float32))
    rows = np.arange(0, q, 20)
    u = plan.sph_project(x.cuda(), n_f, f_min, df).cpu().numpy()[rows].astype(np.complex128)
    plan.close()
    want = ref.sph_project(geom.as_dict(), x.double().numpy(), n_f, f_min, df, rows=rows, aperture=ap)
    size = np.linalg.norm(want)
    rounding = np.linalg.norm(want.astype(np.complex64).astype(np.complex128) - want) / size
    e = np.linalg.norm(u - want) / size
    print(f"[gpu] H_sph {n_f} frequencies from {f_min:g}, {image}: rel {e:.3e}, rounding {rounding:.3e}", flush=True)
    assert e < np.hypot(rounding, 5e-9)


@pytest.mark.parametrize("f", [0.02, 3.0])
def test_adjoint_of_one_frequency(f):
    """H_sph^T at one frequency holds u conj(p0) in FP32 and everything else in FP64: with those
    values the exact sums rounded once (5e-9 in quadrature, as above)."""
    from paper_1304_2017_amd.oat import Plan
    shape, q, dx = (33, 37, 40), 200, 0.4
    o = [synth.centred_origin(n, dx) for n in reversed(shape)]
    geom = synth.Geometry(*reversed(shape), dx, *o, synth.fibonacci_sphere(q, 40.0), 256, 0.05, 0.0, 1.5, 1.0)
    plan = Plan(geom, 0, arc_table=False, segment_table=False)
    gd = geom.as_dict()
    u = torch.view_as_complex(torch.randn((q, 1, 2), generator=torch.Generator().manual_seed(5)))
    a = plan.sph_backproject(u.cuda(), f, 0.1)
    assert torch.equal(plan.sph_backproject_noalloc(u.cuda(), f, 0.1, torch.empty_like(a)), a)
    plan.close()
    vox = np.random.default_rng(2).choice(geom.n_vox, 500, replace=False)
    p0 = np.conj(ref.sph_p0(np.array([f]), gd))
    held = (u.numpy().astype(np.complex128) * p0).astype(np.complex64).astype(np.complex128) / p0
    want = ref.sph_backproject(gd, held, 1, f, 0.1, voxels=vox)
    size = np.linalg.norm(want)
    rounding = np.linalg.norm(want.astype(np.float32) - want) / size
    e = np.linalg.norm(a.cpu().numpy().ravel()[vox] - want) / size
    print(f"[gpu] H_sph^T at {f:g} MHz: rel {e:.3e}, rounding {rounding:.3e}", flush=True)
    assert e < np.hypot(rounding, 5e-9)
