"""Retractions from d = 1024 on whose second iteration is a correction in one term: steps that end with it, just do not (the third takes
the full product up again, as does what a row of R longer than one is cut off at), and end with the first, with the orthogonality figure
and the bf16 copy.  Against the exact Cayley transform in 64 bits on the device."""
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _problem(d, size, sparse):
    g = torch.Generator(device="cuda").manual_seed(d + sparse)
    R = torch.linalg.qr(torch.randn((d, d), generator=g, device="cuda", dtype=torch.float64))[0].float().contiguous()
    G = torch.randn((d, d), generator=g, device="cuda")
    if sparse:  # nearly rank two
        G[:, ::97] *= 300.0
    K = G.double() @ R.double().T.contiguous()
    lr = 2.0 * size / torch.linalg.matrix_norm(K - K.T, 2).item()
    return R, G, lr


def _exact(R, G, lr):
    K = G.double() @ R.double().T.contiguous()
    a = 0.5 * lr * (K - K.T)
    return torch.linalg.solve(torch.eye(len(R), device="cuda", dtype=torch.float64) + a, R.double() - a @ R.double())


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("d,size", [(1024, 1e-9), (1152, 1e-3), (1024, 8e-3), (1408, 2e-2), (2048, 5e-2), (1152, 0.2)])
def test_step(d, size, sparse):
    R, G, lr = _problem(d, size, sparse)
    want = _exact(R, G, lr)
    new, low = R.clone(), torch.empty((d, d), dtype=torch.bfloat16, device="cuda")
    info, err = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")
    kt.kt_cayley_step(new, G, lr, R_lowp=low, info=info, ortho_err=err)
    assert info.item() >= 1 and err.item() < 1e-6
    assert torch.equal(low, new.bfloat16())
    # accepted where four times the distance to the limit, estimated from the changes, is below 3e-7; of a nearly low-rank B the changes
    # alternate between two levels and two of them give a ratio up to four times too small; R is rounded to fp32 once
    assert (new.double() - want).abs().max() <= 3e-7 + 2.0 ** -24 * want.abs().max()
    if size <= 1e-3:
        assert (new.double() - want).norm() <= 2e-7 * d ** 0.5


def test_rows_longer_than_one():
    """R four times an orthogonal matrix: D_1 is longer than its head's exponent allows for, the step is the same linear map."""
    R, G, _ = _problem(1024, 1e-2, False)
    R = (4.0 * R).contiguous()
    K = G.double() @ R.double().T.contiguous()
    lr = 2.0 * 0.05 / torch.linalg.matrix_norm(K - K.T, 2).item()
    new, info = R.clone(), torch.zeros(1, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(new, G, lr, info=info)
    assert info.item() >= 1
    assert (new.double() - _exact(R, G, lr)).norm() <= 4e-6 * 1024 ** 0.5
