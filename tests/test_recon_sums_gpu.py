"""The reconstructions' vector kernels (FP64 inner products, total variation with gradient,
weights and curvature) against the same formulas in FP64: volumes of one voxel, of one-voxel axes,
smaller and larger than the grid.  FP32 terms of a gradient carry a few units of 2^-24 each and
are at most 1: 3e-6; the weights and the sums of FP32 terms are as exact as a term: 1e-6; inner
products are FP64: 1e-13 of the sum of magnitudes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 5, 3), (7, 1, 130), (3, 64, 1), (33, 20, 65),
                                   (80, 71, 90)])
def test_sums_match_fp64(shape):
    import torch
    from paper_1304_2017_amd import recon
    gen = torch.Generator().manual_seed(sum(shape))
    a, d = (torch.randn(shape, generator=gen).cuda() for _ in range(2))
    eps = 0.1
    tv, grad, w, (ad, dd) = recon._tv_sums(a, eps, (a, d), (d, d))
    tv64, grad64, w64 = recon.tv_eps(a.double(), eps)
    assert abs(tv - tv64) <= 1e-6 * tv64
    assert float((grad.double() - grad64).abs().max()) <= 3e-6
    assert float(((w.double() - w64) / w64).abs().max()) <= 1e-6
    a64, d64 = a.double(), d.double()
    assert abs(ad - float((a64 * d64).sum())) <= 1e-13 * float((a64 * d64).abs().sum())
    assert abs(dd - float((d64 * d64).sum())) <= 1e-13 * dd
    hh, slope, curv = recon._step_sums(a, d, a, w)
    c64 = sum((x * x for x in recon.forward_diff(d64)))
    want = float((w.double() * c64).sum())
    assert hh == recon._dot(a, a) and slope == ad
    assert abs(curv - want) <= 1e-6 * want
    tv2, grad2, w2, _ = recon._tv_sums(a, eps)      # fixed order: the same bits again
    assert tv2 == tv and torch.equal(grad2, grad) and torch.equal(w2, w)


def test_other_tensors_take_the_general_path():
    import torch
    from paper_1304_2017_amd import recon
    a = torch.randn((6, 5, 4), device="cuda")
    t = a.transpose(0, 2)
    assert recon._fused(a) and not recon._fused(t) and not recon._fused(a.double())
    assert not recon._fused(a.clone().requires_grad_()) and not recon._fused(a[:0])
    assert recon._dot(t, t) == pytest.approx(recon._dot(a, a), rel=1e-13)
    tv, grad, w, _ = recon._tv_sums(t, 0.1)
    ref = recon._tv_sums(t.contiguous(), 0.1)
    assert tv == pytest.approx(ref[0], rel=1e-6)
    assert float((grad - ref[1]).abs().max()) <= 6e-6
