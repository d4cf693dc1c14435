"""The single-pass d = 128 kernel: tiles of 128 tokens dealt to a number of workgroups that follows from batch and token count.
Ragged last tiles, one and several workgroups per problem, rounds that do not fill the chip, padded rows, and workspaces
that hold fewer partial sums.  Against the oracle at the path's bf16 tolerance (dL/dY is rounded to bf16: 2^-9 per entry, times what cancels in
the sum over tokens)."""
import pytest
import torch

import ktgen
import paper_2503_01483_amd as kt
from parity_util import check_loss_grad, gpu_loss_grad, oracle_loss_grad

pytestmark = pytest.mark.gpu
TOL = 2e-2


def _problem(batch, n, pad=0):
    X = torch.stack([ktgen.make_x(n, 128, seed=n + b, outlier_cols=2, outlier_scale=50.0, dtype="bf16") for b in range(batch)])
    R = torch.stack([ktgen.random_orthogonal(128, seed=100 + b) for b in range(batch)])
    if pad:
        wide = torch.full((batch, n, 128 + pad), 3.0, dtype=torch.bfloat16)
        wide[:, :, :128] = X
        X = wide.cuda()[:, :, :128]
    return X, R


@pytest.mark.parametrize("batch,n,pad", [(1, 1, 0), (2, 15, 0), (1, 16, 8), (3, 127, 0), (1, 128, 0), (2, 129, 0), (1, 385, 8), (5, 2000, 0),
                                         (130, 300, 0), (257, 130, 0)])
def test_against_oracle(batch, n, pad):
    X, R = _problem(batch, n, pad)
    g = gpu_loss_grad(X, R)
    pick = sorted({0, batch // 2, batch - 1})
    o = oracle_loss_grad(X.cpu()[pick].contiguous(), R[pick])
    check_loss_grad({k: v[pick] for k, v in g.items()}, o, TOL)
    assert torch.isfinite(torch.from_numpy(g["dR"])).all()


def test_smaller_workspace_fewer_workgroups():
    """Every size down to what one workgroup per problem needs serves; a byte less is refused."""
    X, R = _problem(3, 1500)
    o = oracle_loss_grad(X, R)
    Xd, Rd = X.cuda(), R.cuda()
    full = kt.kt_workspace_bytes(kt.KT_OP_LOSS_GRAD, 3, 1500, 128, kt.KT_BF16)
    least = 256  # the loss partials
    assert full > least
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    for size in (full, full - 1, full // 2, least, least - 1):
        loss, dR = torch.full((3,), float("nan"), device="cuda"), torch.full((3, 128, 128), float("nan"), device="cuda")
        status = kt.lib().kt_kurtosis_loss_grad(Xd.data_ptr(), 128, Rd.data_ptr(), 128, 3, 1500, 128, kt.KT_BF16, kt.KT_F32, 0.0,
                                                loss.data_ptr(), None, dR.data_ptr(), ws.data_ptr(), size,
                                                torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert (status == 0) == (size >= least), (size, status)
        if status == 0:
            check_loss_grad({"loss": loss.cpu().double().numpy(), "row_kurt": None, "dR": dR.cpu().numpy()}, o, TOL)
