"""The learned preconditioner's BF16 pass at working sizes: volumes whose tiles and columns are those
of 128^3 to 256^3 (eight planes a C1 tile, up to 32 planes a column of C2 and C3, several tiles a
gradient workgroup), ragged in every axis.  Forward: boxes across the borders of tiles, columns and
volume against PyTorch in FP64 with the same roundings; gradients: the whole volume.  Gates as for
the small volumes (test_net_gpu)."""
import os
import re

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_1304_2017_amd import precond
from test_net_gpu import _bf, _conv, _corr, _rel

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _dispatch(d, h, w):
    """Planes of a C1 tile, of a column of C2 and of C3, and tiles per gradient workgroup, with the
    thresholds of the source."""
    text = open(os.path.join(ROOT, "paper_1304_2017_amd", "csrc", "oat_net.hip")).read()

    def const(name):
        return int(re.search(r"\b%s = (\d+)" % name, text).group(1))

    def up(n, t):
        return -(-n // t)

    eight = int(re.search(r"up\(d, 8\) >= (\d+) \? go\(net_c1_kernel<8>", text).group(1))
    c1 = 8 if up(w, 32) * up(h, 8) * up(d, 8) >= eight else 4

    def planes(columns, want):
        zr = 32
        while zr > 4 and columns * up(d, zr) < want:
            zr //= 2
        return zr

    c2 = planes(up(w, 32) * up(h, 8), const("C2_WGS"))
    c3 = planes(up(w, 32) * up(h, 16), int(re.search(r"up\(h, C3Y\), d, (\d+)\)", text).group(1)))
    tiles = up(w, 16) * up(h, 8) * up(d, 4)
    return c1, c2, c3, tiles / const("G16_GRID"), tiles / const("G1_GRID")


def _model(seed):
    g = torch.Generator().manual_seed(seed)
    model = precond.Preconditioner(seed=3, init_scale=1.0)
    for b in model.b:
        b.copy_(0.1 * torch.randn(b.shape, generator=g))
    return model, g


def _reference(x, w, bias):
    w2 = w[1].to(torch.bfloat16)
    xr = _bf(x)[None]
    a1 = _bf(F.relu(_conv(xr, w[0]) + bias[0][:, None, None, None]))
    a2 = _bf(F.relu(_conv(a1, w2) + bias[1][:, None, None, None]))
    return xr, a1, a2, _bf(xr + _bf(_conv(a2, w[2]) + bias[2]))[0]


@pytest.mark.parametrize("shape,planes", [((163, 251, 253), (8, 32, 32)), ((70, 250, 225), (8, 8, 16))])
@pytest.mark.parametrize("xdt", [torch.bfloat16, torch.float32])
def test_forward_at_working_sizes(shape, planes, xdt):
    assert _dispatch(*shape)[:3] == planes
    model, g = _model(1)
    x = torch.randn(shape, generator=g).to(xdt)
    z0 = model.forward(x.cuda())
    z = model.forward(x.cuda(), keep=True)
    assert torch.equal(z, z0)
    _, a1, a2 = model._cache
    w = [t.cpu() for t in model.w]
    bias = [t.double().cpu() for t in model.b]
    rng = np.random.default_rng(2)
    corners = [[0, n] for n in shape]
    # the volume's corners, the borders of tiles and columns, anywhere
    at = [(a, b, c) for a in corners[0] for b in corners[1] for c in corners[2]]
    at += [(8, 8, 32), (16, 16, 64), (32, 32, 96), (64, 128, 128), (shape[0] // 32 * 32, 248, 224)]
    at += [tuple(int(rng.integers(0, n)) for n in shape) for _ in range(12)]
    num, den = np.zeros(3), np.zeros(3)
    for c in at:
        lo = [max(0, v - 5) for v in c]
        hi = [min(n, v + 5) for v, n in zip(c, shape)]
        el = [max(0, v - 3) for v in lo]            # the layers together reach three voxels
        eh = [min(n, v + 3) for v, n in zip(hi, shape)]
        box = tuple(slice(a, b) for a, b in zip(lo, hi))
        inner = tuple(slice(a - e, b - e) for a, b, e in zip(lo, hi, el))
        _, r1, r2, rz = _reference(x[tuple(slice(a, b) for a, b in zip(el, eh))], w, bias)
        for k, (got, want) in enumerate(((z[box], rz[inner]),
                                         (a1[box].permute(3, 0, 1, 2), r1[(slice(None),) + inner]),
                                         (a2[box].permute(3, 0, 1, 2), r2[(slice(None),) + inner]))):
            dif = got.double().cpu() - want
            num[k] += float((dif ** 2).sum())
            den[k] += float((want ** 2).sum())
            assert float(dif.abs().max()) <= 0.05 * float(want.abs().max()), (c, k)
    e = np.sqrt(num / den)
    print(f"[gpu] network {shape} {xdt}: z {e[0]:.1e} a1 {e[1]:.1e} a2 {e[2]:.1e}", flush=True)
    assert e.max() < 2e-3


def test_gradients_at_working_sizes():
    shape = (90, 101, 117)
    d = _dispatch(*shape)
    assert d[3] > 2 and d[4] > 1.5        # the workgroups take up to four and two tiles
    model, g = _model(4)
    x = torch.randn(shape, generator=g).to(torch.bfloat16)
    dz = torch.randn(shape, generator=g).to(torch.bfloat16)
    model.forward(x.cuda(), keep=True)
    grads = model.backward(dz.cuda())
    w = [t.cpu() for t in model.w]
    bias = [t.double().cpu() for t in model.b]
    xr, a1, a2, _ = _reference(x, w, bias)
    d3 = dz.double()[None]
    d2 = _bf(_conv(d3, precond.flip_transpose(w[2])) * (a2 > 0))
    d1 = _bf(_conv(d2, precond.flip_transpose(w[1].to(torch.bfloat16))) * (a1 > 0))
    want = [_corr(xr, d1), _corr(a1, d2), _corr(a2, d3), d1.sum((1, 2, 3)), d2.sum((1, 2, 3)), d3.sum((1, 2, 3))]
    e = [_rel(a, b) for a, b in zip(grads, want)]
    print(f"[gpu] network gradients {shape}: " + " ".join("%.1e" % v for v in e), flush=True)
    # a sum of n products of random sign is held to the size of its terms (sqrt(n) of them would be the
    # sum's own size, and the flips of roundings are independent): as in test_net_gpu for the biases
    scale = [1.0] * 3 + [float(t.abs().sum((1, 2, 3)).norm() / t.sum((1, 2, 3)).norm()) for t in (d1, d2, d3)]
    for v, s, gate in zip(e, scale, [2e-3] * 5 + [1e-5]):
        assert v < gate * max(1.0, s), e
    for a, b in zip(grads, model.backward(dz.cuda())):
        assert torch.equal(a, b)
