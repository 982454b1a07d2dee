"""H_sph over so many transducers that their interval moments are formed in batches: rows on both
sides of the batches' ends against FP64 (gate 5e-7, as for the other interval paths), the same bits
again, and a workspace that does not grow with the transducers."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1304_2017_amd import synth

pytestmark = pytest.mark.gpu


def test_forward_batches_of_transducers():
    from paper_1304_2017_amd.oat import Plan
    shape, q, dx, n_f = (20, 20, 20), 25000, 0.4, 64
    df = 34.0 / n_f
    o = synth.centred_origin(20, dx)
    geom = synth.Geometry(*shape, dx, o, o, o, synth.fibonacci_sphere(q, 60.0), 16, 0.5, 30.0, 1.5, 1.0)
    plan = Plan(geom, 0, arc_table=False, segment_table=False)
    rng = np.random.default_rng(6)
    x = torch.from_numpy((rng.normal(size=shape) * (rng.random(shape) < 0.05)).astype(np.float32))
    u = torch.empty((q, n_f), dtype=torch.complex64, device="cuda")
    xd = x.cuda()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    u = plan.sph_project(xd, n_f, df, df)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    print(f"[gpu] H_sph of {q} transducers: {used / 2**20:.0f} MiB", flush=True)
    assert used < (1 << 30) + (64 << 20)
    assert torch.equal(plan.sph_project(xd, n_f, df, df), u)
    plan.close()
    # a row is at least 6 moments of 8 bytes in some thousand intervals: the batches end near
    # multiples of 2^30 / (48 n); rows from everywhere, close to each other around there
    rows = np.unique(np.concatenate([np.arange(0, q, 97), np.arange(8000, 11000, 13), [q - 1]]))
    want = ref.sph_project(geom.as_dict(), x.double().numpy(), n_f, df, df, rows=rows[::6])
    got = u.cpu().numpy()[rows[::6]]
    e = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
    print(f"[gpu] H_sph of {q} transducers, {len(want)} rows: rel {e.max():.3e}", flush=True)
    assert e.max() < 5e-7
