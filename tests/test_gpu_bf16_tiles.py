"""bf16 loss + gradient with either tile in either product (128 x 128 where tiles are few, 256 x 256 else), d a multiple of 128
but not of 256 among them: the last tile is half empty, and X is read in place by the gradient product.  Against the
same quantities in 64 bits on the device (Eq. 3 and its gradient).  With kept and with recomputed Y the bits are the same."""
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu

# n: one token, edges of 64 / 128 / 256 tokens, ragged ends; d: either side of the rules of both products
SHAPES = [(1, 384, 1), (2, 256, 127), (1, 640, 129), (1, 384, 4097), (3, 512, 300), (1, 1152, 2100), (1, 1664, 9001), (1, 2048, 8000),
          (1, 2688, 3001), (1, 2944, 1025), (2, 1408, 7000)]


def _reference(x, R, pooled):
    y = x @ R
    if pooled:
        i = torch.rsqrt((y * y).mean(1, keepdim=True))
        z = y * i
        c = z - z.mean()
        m2, m3, m4 = (c ** 2).mean(), (c ** 3).mean(), (c ** 4).mean()
        kappa = m4 / m2 ** 2
        s = 1.0 if kappa > 1.8 else -1.0
        g = s * 4.0 / (z.numel() * m2 ** 2) * (c ** 3 - m3 - kappa * m2 * c)
        return (kappa - 1.8).abs(), None, x.T.contiguous() @ (i * (g - z * (z * g).mean(1, keepdim=True)))
    c = y - y.mean(1, keepdim=True)
    m2, m3, m4 = ((c ** k).mean(1, keepdim=True) for k in (2, 3, 4))
    kappa = m4 / m2 ** 2
    G = 4.0 / y.numel() / m2 ** 2 * (c ** 3 - m3 - kappa * m2 * c)
    return kappa.mean(), kappa[:, 0], x.T.contiguous() @ G


@pytest.mark.parametrize("pooled", [False, True])
@pytest.mark.parametrize("batch,d,n", SHAPES)
def test_tiles(batch, d, n, pooled):
    g = torch.Generator(device="cuda").manual_seed(d + n)
    X = torch.randn((batch, n, d + 8), generator=g, device="cuda")
    X[:, :, ::37] *= 20.0
    X = (X + 0.5).bfloat16()[:, :, :d]
    R = torch.linalg.qr(torch.randn((batch, d, d), generator=g, device="cuda"))[0].contiguous()
    out = []
    for recompute in (False, True):
        dR = torch.full((batch, d, d), float("nan"), device="cuda")
        if pooled:
            loss, kurt = kt.kt_pooled_kurtosis_loss_grad(X, R, dR=dR, recompute=recompute), None
        else:
            kurt = torch.empty((batch, n), device="cuda")
            loss = kt.kt_kurtosis_loss_grad(X, R, row_kurt=kurt, dR=dR, recompute=recompute)
        out.append((loss.clone(), kurt, dR))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][2], out[1][2])
    loss, kurt, dR = out[0]
    for b in range(batch):
        l, k, G = _reference(X[b].double(), R[b].bfloat16().double(), pooled)
        # fp32 sums of d products and of row moments: far below 1e-4 of a kurtosis of order one; dL/dY is rounded to bf16
        # (2^-9 of each entry) before the last product
        assert abs(loss[b].double() - l) <= 1e-4 * (l + 1.8)
        if k is not None:
            assert ((kurt[b].double() - k).abs() <= 1e-4 * k).all()
        assert (dR[b].double() - G).norm() <= 2.0 ** -8 * G.norm()


@pytest.mark.parametrize("batch,n,d", [(1, 65, 256), (2, 67, 384), (1, 129, 4096), (1, 500, 1024), (1, 512, 4096), (1, 513, 4096)])
def test_rotated_rows_of_few_tiles(batch, n, d):
    """64 x 64 tiles of bf16 rows, on either side of their last size; fp32 sums of d exact products."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn((batch, n, d + 8), generator=g, device="cuda").bfloat16()[:, :, :d]
    R = torch.randn((batch, d, d), generator=g, device="cuda") * d ** -0.5
    Y = torch.full((batch, n, d), float("nan"), device="cuda")
    kt.kt_rotate_quant_metrics(X, R, Y=Y)
    for b in range(batch):
        x, r = X[b].double(), R[b].bfloat16().double()
        assert ((Y[b].double() - x @ r).abs() <= d * 2.0 ** -24 * (x.abs() @ r.abs())).all()
