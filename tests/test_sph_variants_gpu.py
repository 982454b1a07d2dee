"""H_sph and H_sph^T by their kernels' variants.  H_sph: the variants of its list, moment and synthesis kernels: voxel counts around the list from
one workgroup (8192) and the moments' two block sizes (24576 terms), frequency counts around the
shares of a wave (16, 32) and the frequencies a lane takes (64, 128), block counts around the
waves of a block (256, 768, 2048).  H_sph^T: frequency counts around those that the table kernel takes in one
group of threads, in four, and with the basis from a launch of its own (32, 512), transducer counts
around the slices of 4 to 8.  Sampled rows and voxels against FP64 at 5e-7, the gate of the other
interval-polynomial tests, and the same bits again."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,q,n_f,f_min,df", [
    ((32, 16, 16), 3, 15, 0.4, 0.3), ((32, 16, 16), 1100, 16, 0.3, 0.3), ((11, 27, 28), 600, 17, 0.3, 0.25),
    ((33, 16, 16), 5, 1, 2.0, 0.1), ((24, 32, 32), 40, 31, 0.2, 0.15), ((25, 32, 32), 40, 32, 0.2, 0.15),
    ((20, 20, 20), 1100, 33, 0.2, 0.1),
    ((13, 12, 12), 255, 40, 0.2, 0.1), ((13, 12, 12), 384, 70, 0.2, 0.05), ((12, 12, 12), 520, 9, 0.0, 0.4), ((12, 12, 12), 1030, 20, 0.0, 0.2),
    # two and four frequencies a lane, ragged in the last block
    ((14, 12, 10), 1100, 100, 0.05, 0.05), ((14, 12, 10), 600, 257, 0.02, 0.02), ((9, 8, 7), 2048, 65, 0.1, 0.05)])
def test_variants(shape, q, n_f, f_min, df):
    from paper_1304_2017_amd.oat import Plan
    dx = 0.4
    o = [synth.centred_origin(n, dx) for n in reversed(shape)]
    geom = synth.Geometry(*reversed(shape), dx, *o, synth.fibonacci_sphere(q, 40.0), 256, 0.05, 0.0, 1.5, 1.3)
    plan = Plan(geom, 0, arc_table=False, segment_table=False)
    rng = np.random.default_rng(q + n_f)
    rows = np.unique(np.concatenate([[0, q - 1], rng.integers(0, q, 6)]))
    for keep in (1.0, 0.03):
        x = torch.from_numpy((rng.normal(size=shape) * (rng.random(shape) < keep)).astype(np.float32))
        u = plan.sph_project(x.cuda(), n_f, f_min, df)
        want = ref.sph_project(geom.as_dict(), x.double().numpy(), n_f, f_min, df, rows=rows)
        e = np.linalg.norm(u.cpu().numpy()[rows] - want) / np.linalg.norm(want)
        print(f"[gpu] H_sph {shape}/{q}/{n_f}, {keep:g} set: rel {e:.3e}", flush=True)
        assert e < 5e-7
        assert torch.equal(plan.sph_project(x.cuda(), n_f, f_min, df), u)
    plan.close()


@pytest.mark.parametrize("shape,q,n_f,f_min", [
    ((12, 12, 12), 64, 16, 0.3), ((12, 12, 12), 65, 31, 0.0), ((13, 20, 17), 16, 32, 0.1), ((20, 13, 17), 3, 33, 0.1),
    ((16, 16, 16), 5, 512, 0.0), ((16, 16, 16), 5, 513, 0.0), ((30, 33, 20), 130, 40, 0.2), ((9, 40, 12), 200, 100, 0.0)])
def test_adjoint_variants(shape, q, n_f, f_min):
    from paper_1304_2017_amd.oat import Plan
    dx, df = 0.4, 5.0 / n_f
    o = [synth.centred_origin(n, dx) for n in reversed(shape)]
    geom = synth.Geometry(*reversed(shape), dx, *o, synth.fibonacci_sphere(q, 40.0), 256, 0.05, 0.0, 1.5, 1.3)
    plan = Plan(geom, 0, arc_table=False, segment_table=False)
    u = torch.view_as_complex(torch.randn((q, n_f, 2), generator=torch.Generator().manual_seed(n_f))).cuda()
    a = plan.sph_backproject(u, f_min, df)
    out = torch.full_like(a, float("nan"))
    assert torch.equal(plan.sph_backproject_noalloc(u, f_min, df, out), a)
    plan.close()
    vox = np.random.default_rng(q).choice(geom.n_vox, 60, replace=False)
    want = ref.sph_backproject(geom.as_dict(), u.cpu().numpy().astype(np.complex128), n_f, f_min, df, voxels=vox)
    e = np.linalg.norm(a.cpu().numpy().ravel()[vox] - want) / np.linalg.norm(want)
    print(f"[gpu] H_sph^T {shape}/{q}/{n_f}: rel {e:.3e}", flush=True)
    assert e < 5e-7
