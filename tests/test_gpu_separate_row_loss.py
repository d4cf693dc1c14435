"""Row loss and gradient of bf16 activations where the forward product, the row statistics and dL/dY are launches of their own: fewer than 64 tokens, wide
rows of up to 256, a second round of large tiles for few row blocks, d > 8192 (both tile sizes).  Y kept and Y recomputed: the same bits."""
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 384), (1, 63, 512), (3, 21, 1152), (1, 200, 2688), (2, 128, 4096), (1, 10007, 2048), (1, 300, 8320), (1, 1000, 8320)]


@pytest.mark.parametrize("batch,n,d", SHAPES)
def test_kept_and_recomputed_y(batch, n, d):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn((batch, n, d), generator=g, device="cuda")
    X[:, :, :4] *= 50.0
    X = X.bfloat16()
    R = (torch.randn((batch, d, d), generator=g, device="cuda") / d ** 0.5).contiguous()
    out = []
    for recompute in (False, True):
        dR, rk = torch.full((batch, d, d), float("nan"), device="cuda"), torch.full((batch, n), float("nan"), device="cuda")
        kt.kt_profile_enable(8)
        try:
            kt.kt_profile_reset()
            loss = kt.kt_kurtosis_loss_grad(X, R, dR=dR, row_kurt=rk, recompute=recompute)
            assert kt.kt_profile_read(1)[1] == 1  # dL/dY is a launch of its own
        finally:
            kt.kt_profile_enable(0)
        out.append((loss, rk, dR))
    for a, b in zip(*out):
        assert torch.equal(a, b) and bool(torch.isfinite(a).all())
    # without a gradient the row statistics are the same launches
    only = torch.empty((batch, n), device="cuda")
    assert torch.equal(kt.kt_kurtosis_loss_grad(X, R, row_kurt=only), out[0][0]) and torch.equal(only, out[0][1])


@pytest.mark.parametrize("n,d", [(63, 512), (200, 2688)])
@pytest.mark.parametrize("recompute", [False, True])
def test_against_the_oracle(n, d, recompute):
    X = ktgen.make_x(n, d, seed=5, outlier_cols=4, outlier_scale=50.0, t_frac=0.05, dtype="bf16").reshape(1, n, d).cuda()
    R = ktgen.random_orthogonal(d, seed=6).reshape(1, d, d).cuda()
    dR = torch.empty((1, d, d), device="cuda")
    loss = kt.kt_kurtosis_loss_grad(X, R, dR=dR, recompute=recompute)
    o = oracle.loss_grad(ktgen.to_f64(X[0].cpu()), ktgen.to_f64(ktgen.bf16_round(R[0].cpu())))
    assert abs(loss.item() - o["loss"]) <= 1e-5 * o["loss"]
    want = torch.from_numpy(o["dR"])
    assert (dR[0].cpu().double() - want).norm() <= 6e-3 * want.norm()  # dL/dY is rounded to bf16 (2^-9 an entry)
