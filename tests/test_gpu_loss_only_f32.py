"""fp32 loss without a gradient: on short rows the row moments come out of the product's epilogue, elsewhere from rows of Y.  Sizes on
either side of that rule, wide and unaligned rotations, several problems; and rows of 128 values, which take half a wave each.  Against the same quantities
in 64 bits on the device."""
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _problem(batch, n, d, pad=0):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn((batch, n, d), generator=g, device="cuda") + 0.3
    X[:, :, ::37] *= 10.0
    R = (torch.randn((batch, d, d + pad), generator=g, device="cuda") * d ** -0.5)[:, :, :d]
    return X, R


def _moments(X, R):
    y = X.double() @ R.double()
    c = y - y.mean(1, keepdim=True)
    return y, c, [(c ** k).mean(1, keepdim=True) for k in (2, 3, 4)]


@pytest.mark.parametrize("batch,n,d,pad", [(1, 16256, 128, 0), (1, 16300, 128, 4), (1, 16300, 128, 1), (40, 300, 128, 4), (130, 400, 128, 0), (1, 8100, 256, 0),
                                           (1, 8129, 256, 8), (3, 3000, 256, 4), (1, 8193, 384, 0), (1, 12001, 384, 0), (1, 13000, 512, 0),
                                           (2, 20000, 640, 4)])
@pytest.mark.parametrize("target", [0.0, 1.8])
def test_row_loss(batch, n, d, pad, target):
    X, R = _problem(batch, n, d, pad)
    kurt = torch.full((batch, n), float("nan"), device="cuda")
    loss = kt.kt_kurtosis_loss_grad(X, R, kappa_target=target, row_kurt=kurt)
    for b in {0, batch - 1}:
        _, _, (m2, _, m4) = _moments(X[b], R[b])
        kappa = (m4 / m2 ** 2)[:, 0]
        want = kappa.mean() if target == 0.0 else (kappa - target).abs().mean()
        # y errs by about sqrt(d) 2^-24 of its size, a kurtosis by four times that
        assert ((kurt[b].double() - kappa).abs() / kappa).max().item() <= 1e-5
        assert abs(loss[b].item() - want.item()) <= 1e-5 * (want.item() + target)


@pytest.mark.parametrize("batch,n,d", [(1, 20000, 128), (2, 9000, 256), (1, 300, 128), (3, 1000, 128)])
def test_pooled_loss_and_gradient(batch, n, d):
    X, R = _problem(batch, n, d)
    kappa, dR = torch.empty(batch, device="cuda"), torch.full((batch, d, d), float("nan"), device="cuda")
    only = kt.kt_pooled_kurtosis_loss_grad(X, R, kappa=kappa)
    loss = kt.kt_pooled_kurtosis_loss_grad(X, R, dR=dR)
    for b in {0, batch - 1}:
        y = X[b].double() @ R[b].double()
        i = torch.rsqrt((y * y).mean(1, keepdim=True))
        z = y * i
        c = z - z.mean()
        m2, m3, m4 = ((c ** k).mean() for k in (2, 3, 4))
        k = m4 / m2 ** 2
        g = torch.sign(k - 1.8) * 4.0 / (z.numel() * m2 ** 2) * (c ** 3 - m3 - k * m2 * c)
        want = X[b].double().T.contiguous() @ (i * (g - z * (z * g).mean(1, keepdim=True)))
        assert abs(kappa[b].item() - k.item()) <= 1e-5 * k.item()
        for got in (only, loss):
            assert abs(got[b].item() - abs(k.item() - 1.8)) <= 1e-5 * k.item()
        assert ((dR[b].double() - want).norm() / want.norm()).item() <= 1e-5


@pytest.mark.parametrize("batch,n", [(1, 1), (2, 7), (1, 129), (64, 1000), (1, 70001)])
def test_rows_of_128_values(batch, n):
    X, R = _problem(batch, n, 128)
    dR, kurt = torch.full((batch, 128, 128), float("nan"), device="cuda"), torch.full((batch, n), float("nan"), device="cuda")
    loss = kt.kt_kurtosis_loss_grad(X, R, row_kurt=kurt, dR=dR)
    for b in {0, batch - 1}:
        y, c, (m2, m3, m4) = _moments(X[b], R[b])
        kappa = m4 / m2 ** 2
        want = X[b].double().T.contiguous() @ (4.0 / y.numel() / m2 ** 2 * (c ** 3 - m3 - kappa * m2 * c))
        assert ((kurt[b].double() - kappa[:, 0]).abs() / kappa[:, 0]).max().item() <= 1e-5
        assert abs(loss[b].item() - kappa.mean().item()) <= 1e-5 * kappa.mean().item()
        assert ((dR[b].double() - want).norm() / want.norm()).item() <= 1e-5
