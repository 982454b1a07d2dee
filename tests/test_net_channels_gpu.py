"""The learned preconditioner in BF16 storage with other layers than the 16-channel ones of the
whole-network kernels: one channel throughout, 16 -> 1 -> 1, no bias, and channel counts that no
kernel has.  They go layer by layer, against PyTorch in FP64 with the same roundings to BF16 (sums
of at most 432 FP32 products before each rounding to 2^-9: gate 1e-2)."""
import pytest
import torch
import torch.nn.functional as F

from paper_1304_2017_amd import oat, precond

pytestmark = pytest.mark.gpu


class OneChannel(precond.Preconditioner):
    CH = 1


def _model(kind):
    if kind == "one":
        return OneChannel(seed=2, init_scale=1.0)
    model = precond.Preconditioner(seed=2, init_scale=1.0)
    if kind == "mixed":
        model.w[1], model.b[1] = model.w[1][:1].clone(), model.b[1][:1].clone()
        model.w[2] = model.w[2][:, :1].clone()
    elif kind == "no bias":
        model.b = [None, None, None]
    return model


@pytest.mark.parametrize("kind", ["one", "mixed", "no bias"])
def test_other_layers(kind):
    model = _model(kind)
    g = torch.Generator().manual_seed(4)
    x = torch.randn((9, 11, 21), generator=g)
    z = model.forward(x.cuda(), keep=True)

    def bf(t):
        return t.to(torch.bfloat16).double()

    def conv(a, k):
        w = model.w[k].cpu()
        w = bf(w) if w.shape[0] == w.shape[1] == 16 else w.double()
        b = None if model.b[k] is None else model.b[k].double().cpu()
        return F.conv3d(a[None], w.reshape(w.shape[0], w.shape[1], 3, 3, 3), b, padding=1)[0]

    a = bf(x)[None]
    want = bf(a + bf(conv(bf(F.relu(conv(bf(F.relu(conv(a, 0))), 1))), 2)))[0]
    assert float((z.double().cpu() - want).norm() / want.norm()) < 1e-2
    grads = model.backward(torch.randn(x.shape, generator=g).cuda())
    assert [tuple(t.shape) for t in grads[:3]] == [tuple(w.shape) for w in model.w]
    assert all(bool(t.isfinite().all()) for t in grads)


def test_channel_counts_that_no_kernel_has():
    class Eight(precond.Preconditioner):
        CH = 8

    with pytest.raises(oat.OatError):
        Eight(seed=2).forward(torch.zeros((4, 4, 4), device="cuda"))


def test_layers_that_change_between_the_passes():
    model = precond.Preconditioner(seed=2)
    x = torch.zeros((4, 4, 4), device="cuda")
    model.forward(x, keep=True)
    model.w[1] = model.w[1][:1].clone()
    with pytest.raises(ValueError):
        model.backward(x)
