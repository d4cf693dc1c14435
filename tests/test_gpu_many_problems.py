"""More rotations than 32 bits count threads for: R is written transposed by batch (d / 64)^2 workgroups of 256 threads, which from 64 GiB of
bf16 R on are more than 2^31.  A loss without a gradient, which has nothing else to clear or to write between the problems; a few
problems have values, at both ends and where the count passes 2^31, all others are zero rows without spread."""
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def test_loss_of_more_than_2_31_transposing_threads():
    d, n = 768, 2
    batch = 2 ** 23 // (d // 64) ** 2 + 2
    assert batch * (d // 64) ** 2 * 256 > 2 ** 31
    need = kt.kt_workspace_bytes(kt.KT_OP_LOSS_GRAD_RECOMPUTE, batch, n, d, kt.KT_BF16)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < need + 2 * batch * d * d + 2 ** 33:
        pytest.skip("needs about 140 GB of device memory")
    R = torch.zeros((batch, d, d), dtype=torch.bfloat16, device="cuda")
    X = torch.zeros((batch, n, d), dtype=torch.bfloat16, device="cuda")
    used = (0, 1, batch // 2, batch - 2, batch - 1)
    for b in used:
        R[b] = ktgen.random_orthogonal(d, seed=b).bfloat16().cuda()
        X[b] = ktgen.make_x(n, d, seed=b, outlier_cols=3, outlier_scale=30.0, dtype="bf16").cuda()
    kurt = torch.full((batch, n), float("nan"), device="cuda")
    loss = torch.full((batch,), float("nan"), device="cuda")
    kt.kt_kurtosis_loss_grad(X, R, loss=loss, row_kurt=kurt, recompute=True)
    for b in used:
        o = oracle.loss_grad(ktgen.to_f64(X[b].cpu()), ktgen.to_f64(R[b].cpu()), want_dR=False)
        assert abs(loss[b].item() - o["loss"]) <= 1e-5 * o["loss"]
        loss[b], kurt[b] = 0.0, 0.0
    assert bool((loss == 0).all()) and bool((kurt == 0).all())
    del R, X
    torch.cuda.empty_cache()
