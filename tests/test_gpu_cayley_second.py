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


@pytest.mark.parametrize("norm", [2.0, 128.0])
def test_rows_far_longer_than_one(norm):
    """A B of rank two along a column of R times a Hadamard matrix: every product of D_1 = -2 R B^T has the same sign, so that its head meets its
    bound, and with rows of norm 128 is cut off.  The change of the second iteration is small enough to end with, were it not for that."""
    d, half = 1024, 2.0 ** -15
    H = torch.ones((1, 1), device="cuda", dtype=torch.float64)
    while len(H) < d:
        H = torch.cat([torch.cat([H, H], 1), torch.cat([H, -H], 1)], 0)
    R = (H * (norm / d ** 0.5)).float().contiguous()
    # G R^T = e_1 1^T: B has 2^-15 in its first row and column.  Powers of two everywhere: the products and their sums are exact
    K = torch.zeros((d, d), device="cuda", dtype=torch.float64)
    K[0] = 1.0
    G = (K @ R.double() / norm ** 2).float().contiguous()
    new, info = R.clone(), torch.zeros(1, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(new, G, 2 * half, info=info)
    assert info.item() >= 2
    want = _exact(R, G, 2 * half)
    # accepted within 3e-7 of the limit, R rounded to fp32 once, 22 bits of U
    off = (new.double() - want).abs().max().item()
    assert off <= 3e-7 + 2.0 ** -24 * want.abs().max() + 2.0 ** -21 * (want - R.double()).abs().max(), off
