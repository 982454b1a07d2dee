"""H_sph and H_sph^T on the interval polynomials (the path of larger problems), at the sizes where
its pieces can go wrong: ragged voxel tiles, frequency counts around the blocks of 64, 128 and 256,
zero and narrow bands, transducers at different distances, finite faces, images with few or no
voxels set, more tiles than one pass takes and more tables than one batch holds.

Gate 5e-7: outputs and tables are rounded to FP32 (6e-8 a value; up to 8 table coefficients of a
value add in quadrature, and a node evaluates 7 FP32 multiply-adds), the polynomials' own errors
are below 4e-8, and the sums are FP64 or integers."""
import numpy as np
import pytest
import torch  # before the library: one HIP runtime for both

from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu
GATE = 5e-7


def _geom(nx, ny, nz, q, dx=0.4, rs=40.0, spread=0.0):
    xyz = synth.fibonacci_sphere(q, rs) * (1.0 + spread * np.arange(q)[:, None] / q)
    return synth.Geometry(nx, ny, nz, dx, synth.centred_origin(nx, dx), synth.centred_origin(ny, dx),
                          synth.centred_origin(nz, dx), xyz, 256, 0.05, 0.0, 1.5, 1.3)


def _plan(geom):
    from paper_1304_2017_amd.oat import Plan
    return Plan(geom, 0, arc_table=False, segment_table=False)


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("shape,q,n_f,f_min,df,faces,spread", [
    ((17, 16, 9), 7, 65, 0.0, 0.05, 0, 0.0),
    ((16, 33, 8), 5, 64, 0.3, 0.02, 2, 0.0),
    ((31, 15, 17), 9, 129, 0.04, 0.04, 0, 0.7),
    ((20, 20, 20), 3, 256, 0.0, 0.02, 0, 0.0),
    ((20, 21, 19), 300, 257, 0.02, 0.02, 0, 0.0),
    ((24, 20, 20), 6, 16, 4.7, 0.02, 3, 0.1),
    ((40, 40, 12), 2100, 17, 0.0, 0.01, 0, 0.0)])
def test_interval_polynomials(shape, q, n_f, f_min, df, faces, spread):
    geom = _geom(*shape, q, spread=spread)
    gd = geom.as_dict()
    rng = np.random.default_rng(n_f)
    plan = _plan(geom)
    ap = None
    if faces:
        plan.set_aperture(2.0, 1.5, faces)
        ap = (2.0, 1.5, faces)
    rows = np.unique(rng.integers(0, q, 6))
    for img in (rng.normal(size=geom.shape), rng.normal(size=geom.shape) * (rng.random(geom.shape) < 0.03)):
        x = torch.from_numpy(img.astype(np.float32)).cuda()
        u = plan.sph_project(x, n_f, f_min, df)
        want = ref.sph_project(gd, x.double().cpu().numpy(), n_f, f_min, df, rows=rows, aperture=ap)
        e = _rel(u.cpu().numpy()[rows], want)
        print(f"[gpu] H_sph {shape}/{q}/{n_f}: rel {e:.3e}", flush=True)
        assert e < GATE
        assert torch.equal(plan.sph_project(x, n_f, f_min, df), u)
    y = torch.randn((q, n_f, 2), generator=torch.Generator().manual_seed(n_f))
    y = torch.view_as_complex(y).cuda()
    vox = rng.choice(geom.n_vox, 60, replace=False)
    a = plan.sph_backproject(y, f_min, df)
    want = ref.sph_backproject(gd, y.cpu().numpy().astype(np.complex128), n_f, f_min, df, voxels=vox, aperture=ap)
    e = _rel(a.cpu().numpy().ravel()[vox], want)
    print(f"[gpu] H_sph^T {shape}/{q}/{n_f}: rel {e:.3e}", flush=True)
    assert e < GATE
    out = torch.empty_like(a)
    assert torch.equal(plan.sph_backproject_noalloc(y, f_min, df, out), a)
    plan.close()


def test_zero_and_non_finite_images():
    geom = _geom(20, 20, 20, 4)
    plan = _plan(geom)
    x = torch.zeros(geom.shape, device="cuda")
    assert float(plan.sph_project(x, 64, 0.0, 0.05).abs().max()) == 0.0
    x[3, 4, 5] = float("inf")
    assert bool(torch.isnan(torch.view_as_real(plan.sph_project(x, 64, 0.0, 0.05))).all())
    x[3, 4, 5] = 1e-38
    x[5, 4, 5] = 1e37
    u = plan.sph_project(x, 64, 0.0, 0.05)
    want = ref.sph_project(geom.as_dict(), x.double().cpu().numpy(), 64, 0.0, 0.05)
    assert _rel(u.cpu().numpy().astype(np.complex128), want) < GATE
    plan.close()


@pytest.mark.parametrize("shape,q,n_f,f_max,dx", [
    ((33, 20, 18), 3000, 64, 50.0, 0.4),        # six batches of tables
    ((16 * 1025, 1, 1), 64, 100, 1.0, 0.004)])  # 1025 tiles: two passes
def test_batches_and_passes(shape, q, n_f, f_max, dx):
    geom = _geom(*shape, q, dx=dx, rs=60.0)
    plan = _plan(geom)
    df = f_max / n_f
    y = torch.randn((q, n_f, 2), generator=torch.Generator().manual_seed(3))
    y = torch.view_as_complex(y).cuda()
    a = plan.sph_backproject(y, 0.0, df)
    vox = np.concatenate([[0, geom.n_vox - 1], np.random.default_rng(0).choice(geom.n_vox, 20, replace=False)])
    want = ref.sph_backproject(geom.as_dict(), y.cpu().numpy().astype(np.complex128), n_f, 0.0, df, voxels=vox)
    e = _rel(a.cpu().numpy().ravel()[vox], want)
    print(f"[gpu] H_sph^T {shape}/{q}/{n_f}: rel {e:.3e}", flush=True)
    assert e < GATE
    out = torch.full_like(a, float("nan"))
    assert torch.equal(plan.sph_backproject_noalloc(y, 0.0, df, out), a)
    plan.close()


def test_forward_over_more_voxels_than_one_pass():
    """2^24 + 65536 voxels, a few of them set on both sides of the first pass's end."""
    geom = _geom(257, 256, 256, 2, dx=0.05)
    plan = _plan(geom)
    x = torch.zeros(geom.shape, device="cuda")
    flat = x.view(-1)
    idx = [0, 123, 1 << 23, (1 << 24) - 1, 1 << 24, geom.n_vox - 1]
    val = [1.0, -2.0, 0.5, 3.0, -1.5, 0.25]
    for i, v in zip(idx, val):
        flat[i] = v
    n_f, f_min, df = 40, 0.1, 0.1
    u = plan.sph_project(x, n_f, f_min, df).cpu().numpy()
    gd = geom.as_dict()
    i = np.array(idx)
    r = np.stack([geom.x0 + geom.dx * (i % 257), geom.y0 + geom.dx * (i // 257 % 256),
                  geom.z0 + geom.dx * (i // (257 * 256))], 1)
    f = f_min + df * np.arange(n_f)
    for q in range(2):
        want = ref.sph_p0(f, gd) * (ref.sph_sir(gd, q, r, f) @ np.array(val))
        e = _rel(u[q], want)
        print(f"[gpu] H_sph 257x256x256 row {q}: rel {e:.3e}", flush=True)
        assert e < GATE
    plan.close()
