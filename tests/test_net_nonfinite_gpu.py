"""The learned preconditioner's BF16 pass on values that are not finite, against its layers one by
one (conv3d, whose products are single FP32 products): every infinity keeps its place and sign and
every NaN its place, in the output, the kept activations and the gradients.  C3's weight gradient is
taken in FP64 over the voxel pairs inside the volume: conv3d_weight_grad also multiplies dz by the
zeros around it, the network's kernels do not."""
import pytest
import torch

from paper_1304_2017_amd import precond

pytestmark = pytest.mark.gpu
SHAPE = (16, 16, 32)     # whole tiles of every kernel, so no layer multiplies zeros beyond the volume


def _corr(x, g):
    """dw[0][ci][t] = sum_v g[0][v] x[ci][v + t - 1] over the v and v + t - 1 inside the volume."""
    out = torch.empty((1, x.shape[0], 27), dtype=torch.float64)
    for t in range(27):
        gs, xs = [0], [slice(None)]
        for o, n in zip((t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1), x.shape[1:]):
            gs.append(slice(max(0, -o), n - max(0, o)))
            xs.append(slice(max(0, o), n - max(0, -o)))
        out[0, :, t] = (x[tuple(xs)].double() * g[tuple(gs)].double()).sum((1, 2, 3)).cpu()
    return out


def _layers(model, x, dz):
    """z, a1, a2 (channel-last) and the gradients, layer by layer in BF16 storage."""
    bf = torch.bfloat16
    x1 = x.to(bf)[None]
    a1 = precond.conv3d(x1, model.w[0], model.b[0], relu=True)
    a2 = precond.conv3d(a1, model.w[1], model.b[1], relu=True)
    z = (x1.float() + precond.conv3d(a2, model.w[2], model.b[2]).float()).to(bf)[0]
    d3 = dz.to(bf)[None]
    dw3, db3 = _corr(a2, d3), precond.conv3d_weight_grad(a2, d3)[1]
    d2 = precond.conv3d(d3, precond.flip_transpose(model.w[2]), None, mask=a2)
    dw2, db2 = precond.conv3d_weight_grad(a1, d2)
    d1 = precond.conv3d(d2, precond.flip_transpose(model.w[1]), None, mask=a1)
    dw1, db1 = precond.conv3d_weight_grad(x1, d1)
    return [z, a1.permute(1, 2, 3, 0), a2.permute(1, 2, 3, 0), dw1, dw2, dw3, db1, db2, db3]


def _same(got, want, what):
    got, want = got.float().cpu(), want.float().cpu()
    assert torch.equal(got.isnan(), want.isnan()), what
    assert torch.equal(got.isinf(), want.isinf()), what
    assert torch.equal(got[got.isinf()], want[want.isinf()]), what
    ok = want.isfinite()
    # BF16 layers whose sums are ordered otherwise: a rounding now and then
    scale = float(want[ok].norm()) if bool(ok.any()) else 0.0
    assert float((got[ok] - want[ok]).norm()) <= 2e-3 * scale, what


@pytest.mark.parametrize("where", ["input", "C1", "C2", "dz"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("at", [(5, 6, 7), (0, 0, 0), (15, 15, 31), (8, 7, 16)])
def test_values_that_are_not_finite(where, value, at):
    g = torch.Generator().manual_seed(7)
    model = precond.Preconditioner(seed=3, init_scale=1.0)
    x = torch.randn(SHAPE, generator=g)
    dz = torch.randn(SHAPE, generator=g)
    if where == "input":
        x[at] = value
    elif where == "dz":
        dz[at] = value
    elif where == "C1":
        # finite inputs whose first layer overflows in one channel around a voxel; the other
        # channels stay far from overflow, so no result depends on the order of a sum
        x[at] = 1e20 if value > 0 else -1e20
        model.w[0][3] *= 1e25
    else:
        # the same in the second layer: one product overflows, the channel's others are zero
        x[at] = 1e15 if value > 0 else -1e15
        model.w[1][3] = 0.0
        model.w[1][3, 2, 13] = 1e30
    x, dz = x.cuda(), dz.cuda()
    want = _layers(model, x, dz)
    z = model.forward(x, keep=True)
    assert torch.equal(model.forward(x).view(torch.int16), z.view(torch.int16))
    got = [z, model._cache[1], model._cache[2]] + model.backward(dz)
    if where != "dz":
        assert any(not bool(t.isfinite().all()) for t in want[:3])
    for a, b, what in zip(got, want, ("z", "a1", "a2", "dw1", "dw2", "dw3", "db1", "db2", "db3")):
        _same(a.reshape(b.shape), b, what)


@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
def test_infinite_weights(value):
    model = precond.Preconditioner(seed=3, init_scale=1.0)
    model.w[0][5, 0, 13] = value
    model.w[2][0, 4, 0] = value
    g = torch.Generator().manual_seed(8)
    x, dz = torch.randn(SHAPE, generator=g).cuda(), torch.randn(SHAPE, generator=g).cuda()
    want = _layers(model, x, dz)
    z = model.forward(x, keep=True)
    for a, b, what in zip([z, model._cache[1], model._cache[2]], want, ("z", "a1", "a2")):
        _same(a, b, what)
