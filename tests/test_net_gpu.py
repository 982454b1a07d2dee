"""The learned preconditioner's BF16 pass (oat_net_forward, oat_net_backward) against PyTorch in
FP64 on the CPU with the same roundings: layer outputs to BF16, C2's weights to BF16.

Both sides then differ by FP32 sums (up to 432 products: below 1e-5 of a value) before each BF16
rounding, which flips a rounding (2^-8 of a value) for at most about 1e-5 * 2^9 of the values: an
L2 difference below 2^-8 * sqrt(5e-3) = 3e-4 a layer, 1e-3 after three.  A gradient is a sum over
voxels of such values: gate 2e-3 (the flips are independent), the last bias, a plain sum of dz, 1e-5."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_1304_2017_amd import oat, precond

pytestmark = pytest.mark.gpu


def _bf(t):
    return t.to(torch.bfloat16).double()


def _conv(x, w):
    return F.conv3d(x[None], w.double().reshape(w.shape[0], w.shape[1], 3, 3, 3), padding=1)[0]


def _corr(x, g):
    """dw[co][ci][t] = sum_v g[co][v] x[ci][v + t - 1]."""
    co, ci = g.shape[0], x.shape[0]
    d, h, w = g.shape[1:]
    p = F.pad(x, (1, 1, 1, 1, 1, 1))
    out = torch.zeros((co, ci, 27), dtype=torch.float64)
    for t in range(27):
        a, b, c = t // 9, t // 3 % 3, t % 3
        out[:, :, t] = torch.einsum("ozyx,izyx->oi", g, p[:, a:a + d, b:b + h, c:c + w])
    return out


def _rel(a, b):
    a, b = a.double().cpu(), b.double()
    return float((a - b).norm() / b.norm().clamp(min=1e-30))


@pytest.mark.parametrize("shape", [(1, 1, 1), (8, 8, 16), (9, 17, 33), (5, 40, 31), (33, 3, 70), (34, 16, 32)])
@pytest.mark.parametrize("xdt", [torch.bfloat16, torch.float32])
def test_network_pass_and_gradients(shape, xdt):
    g = torch.Generator().manual_seed(sum(shape))
    model = precond.Preconditioner(seed=3, init_scale=1.0)
    for b in model.b:
        b.copy_(0.1 * torch.randn(b.shape, generator=g))
    x = torch.randn(shape, generator=g).to(xdt)
    dz = torch.randn(shape, generator=g).to(torch.bfloat16)
    z0 = model.forward(x.cuda())
    z = model.forward(x.cuda(), keep=True)
    assert z.dtype == torch.bfloat16 and torch.equal(z, z0)
    grads = model.backward(dz.cuda())
    w = [t.cpu() for t in model.w]
    bias = [t.double().cpu() for t in model.b]
    xr, w2 = _bf(x)[None], w[1].to(torch.bfloat16)
    a1 = _bf(F.relu(_conv(xr, w[0]) + bias[0][:, None, None, None]))
    a2 = _bf(F.relu(_conv(a1, w2) + bias[1][:, None, None, None]))
    zr = _bf(xr + _bf(_conv(a2, w[2]) + bias[2]))[0]
    d3 = dz.double()[None]
    d2 = _bf(_conv(d3, precond.flip_transpose(w[2])) * (a2 > 0))
    d1 = _bf(_conv(d2, precond.flip_transpose(w2)) * (a1 > 0))
    want = [_corr(xr, d1), _corr(a1, d2), _corr(a2, d3), d1.sum((1, 2, 3)), d2.sum((1, 2, 3)), d3.sum((1, 2, 3))]
    e = [_rel(z, zr)] + [_rel(a, b) for a, b in zip(grads, want)]
    print(f"[gpu] network {shape} {xdt}: " + " ".join("%.1e" % v for v in e), flush=True)
    # cancelling bias sums are held to the size of their terms
    scale = [1.0] * 4 + [float(d.abs().sum((1, 2, 3)).norm() / d.sum((1, 2, 3)).norm()) for d in (d1, d2, d3)]
    assert e[0] < 2e-3
    for v, s, gate in zip(e[1:], scale[1:], [2e-3] * 5 + [1e-5]):
        assert v < gate * max(1.0, s), e
    for a, b in zip(grads, model.backward(dz.cuda())):
        assert torch.equal(a, b)


def test_network_weight_terms_keep_fp32_weights():
    """A 1 -> 16 layer with weights that need more than one BF16 term: the terms' sum must act as the
    FP32 weight (a single term would be off by up to 2^-9)."""
    model = precond.Preconditioner(seed=5)
    g = torch.Generator().manual_seed(1)
    x = torch.zeros((3, 3, 3), dtype=torch.bfloat16)
    x[1, 1, 1] = 1.0
    model.w[0].copy_(1.0 + 2.0 ** -10 * torch.rand((16, 1, 27), generator=g))
    model.b[0].copy_(torch.full((16,), -1.0))
    model.forward(x.cuda(), keep=True)
    a1 = model._cache[1].permute(3, 0, 1, 2).cpu()
    want = (precond.flip_transpose(model.w[0].cpu())[0].reshape(16, 3, 3, 3) - 1.0).to(torch.bfloat16)
    assert torch.equal(a1, want)


def test_network_arguments():
    L = oat.lib()
    assert L.oat_net_workspace(0, 4, 4, 0) == 0
    t = torch.zeros(4096, device="cuda")
    p = precond._ptr(t)
    args = [p] * 10
    assert L.oat_net_forward(p, 7, 4, 4, 4, *args, 1 << 20, None) == oat.OAT_ERR_DTYPE
    assert L.oat_net_forward(None, 0, 4, 4, 4, *args, 1 << 20, None) == oat.OAT_ERR_ARG
    assert L.oat_net_forward(p, 0, 4, 0, 4, *args, 1 << 20, None) == oat.OAT_ERR_ARG
    model = precond.Preconditioner()
    with pytest.raises(ValueError):
        model.forward(torch.zeros((4, 4, 4), device="cuda"), keep=True)
        model.backward(torch.zeros((4, 4, 5), device="cuda"))
    model.w[0] = model.w[0].double()
    with pytest.raises(ValueError):
        model.forward(torch.zeros((4, 4, 4), device="cuda"))
