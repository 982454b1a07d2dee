"""H_sph of an image of one large value among very many small ones: the small ones' terms keep their
bits however many there are (2^22 voxels, 64 face nodes each).  Against FP64 sums over the same
voxels; gate 1e-7 of a row's 2-norm, of which the outputs' rounding to FP32 is 2.5e-8 and the
interval polynomials at most 4e-8."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


def test_one_large_value_among_many():
    from paper_1304_2017_amd.oat import Plan
    n, dx, n_f, f_min, df = 161, 0.05, 3, 0.7, 0.9
    o = synth.centred_origin(n, dx)
    xyz = synth.fibonacci_sphere(256, 30.0)     # as many transducers as take the voxels in one part
    geom = synth.Geometry(n, n, n, dx, o, o, o, xyz, 256, 0.1, 0.0, 1.5, 1.0)
    ap = (1.0, 1.0, 8)
    plan = Plan(geom, 0, arc_table=False, segment_table=False)
    plan.set_aperture(*ap)
    x = 1e-6 * torch.randn((n, n, n), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    x[80, 71, 92] = 1.0
    u = plan.sph_project(x, n_f, f_min, df).cpu().numpy()
    plan.close()
    gd = geom.as_dict()
    f = f_min + df * np.arange(n_f)
    c = o + dx * torch.arange(n, device="cuda", dtype=torch.float64)
    a = x.double()
    for q in (3, 200):
        pts, wts = ref.sph_face_points(gd, q, ap)
        s = torch.zeros(n_f, dtype=torch.complex128, device="cuda")
        for p, w in zip(pts, wts):
            d = torch.sqrt((c - p[2])[:, None, None] ** 2 + (c - p[1])[:, None] ** 2 + (c - p[0]) ** 2)
            t = float(w) * a / (2 * np.pi * d)
            for i in range(n_f):
                ph = 2 * np.pi * torch.remainder(f[i] * d / geom.c0, 1.0)
                s[i] += torch.complex((t * ph.cos()).sum(), -(t * ph.sin()).sum())
        want = ref.sph_p0(f, gd) * s.cpu().numpy()
        e = float(np.linalg.norm(u[q] - want) / np.linalg.norm(want))
        print(f"[gpu] H_sph one of 2^22 voxels, row {q}: rel {e:.3e}", flush=True)
        assert e < 1e-7
