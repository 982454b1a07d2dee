"""Small grids, where G and G^T split their units over workgroups and waves: slices of one
transducer, slices that do not divide the transducers or the windows of 128, units with fewer
segments than parts, one-cell bricks, and transducers so near that ring segments leave a brick and
come back (two table entries).  Against the FP64 oracle at the gates of the other parity
tests (1e-5 in FP32, 5e-7 for G alone; 2e-3 and half a BF16 unit for BF16 storage), and bit for
bit over the table paths for G^T."""
import math

import numpy as np
import pytest

from checks import BF16_ELEM, check
from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


def _geometry(nx, ny, nz, q, dx=0.5, rs=25.0):
    xyz = synth.fibonacci_sphere(q, rs)
    return synth.Geometry(nx, ny, nz, dx, synth.centred_origin(nx, dx), synth.centred_origin(ny, dx),
                          synth.centred_origin(nz, dx), xyz, 256, 0.1, 0.0, 1.5, 1.0,
                          np.full(q, 4 * math.pi * rs * rs / q))


@pytest.mark.parametrize("shape,q,rs", [((20, 20, 20), 1, 25.0), ((1, 2, 3), 3, 25.0),
                                        ((21, 20, 41), 37, 25.0), ((32, 19, 40), 129, 25.0),
                                        ((40, 21, 20), 300, 25.0), ((38, 20, 20), 24, 12.6),
                                        ((20, 20, 20), 40, 9.2)])
def test_small_grids_split_units(shape, q, rs):
    import torch
    from paper_1304_2017_amd.oat import Plan
    geom = _geometry(*shape, q, rs=rs)
    gd = geom.as_dict()
    rng = np.random.default_rng(q)
    img = rng.normal(size=geom.shape).astype(np.float32)
    y = rng.normal(size=(q, geom.n_t)).astype(np.float32)
    plan = Plan(geom, 0)
    assert plan.stats()["segment_table_entries"] > 0
    x, yd = torch.from_numpy(img).cuda(), torch.from_numpy(y).cuda()
    g, p, a = plan.project(x, srt_only=True), plan.project(x), plan.backproject(yd)
    check(f"G {shape}/{q}", g.cpu().numpy(), ref.srt(gd, img.astype(np.float64)), 5e-7)
    check(f"H {shape}/{q}", p.cpu().numpy(), ref.project(gd, img.astype(np.float64)), 1e-5)
    check(f"H^T {shape}/{q}", a.cpu().numpy(), ref.backproject(gd, y.astype(np.float64)), 1e-5)
    xb = x.bfloat16()
    pb = plan.project(xb)
    check(f"H bf16 {shape}/{q}", pb.float().cpu().numpy(),
          ref.project(gd, xb.double().cpu().numpy()), 2e-3, BF16_ELEM)
    for _ in range(2):      # order-independent sums: the same bits again
        assert torch.equal(plan.project(x), p) and torch.equal(plan.backproject(yd), a)
    for tables in (dict(segment_table=0), dict(segment_table=0, arc_table=0)):
        other = Plan(geom, 0, **tables)
        assert torch.equal(other.backproject(yd), a)
        other.close()
    plan.close()


@pytest.mark.parametrize("shape,q", [((181, 200, 163), 320), ((301, 182, 161), 259)])
def test_whole_units_on_node_pairs(shape, q):
    """Grids of whole units, where an FP32 image is read as node pairs and two points at a time: G
    against the table-free walk, each within 5e-7 of the oracle, so 1e-6 apart; edge bricks are
    partly filled and the runs of points even and odd."""
    import torch
    from paper_1304_2017_amd.oat import Plan
    geom = _geometry(*shape, q, dx=0.1, rs=25.0)
    rng = np.random.default_rng(q)
    x = torch.from_numpy(rng.normal(size=geom.shape).astype(np.float32)).cuda()
    plan = Plan(geom, 0)
    assert plan.stats()["segment_table_entries"] > 0
    g = plan.project(x, srt_only=True)
    assert torch.equal(plan.project(x, srt_only=True), g)
    plan.close()
    plain = Plan(geom, 0, segment_table=0, arc_table=0)
    check(f"G {shape}/{q}", g.cpu().numpy(),
          plain.project(x, srt_only=True).double().cpu().numpy(), 1e-6)
    plain.close()
