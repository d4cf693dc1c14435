"""Retractions with products of fp16 heads and tails (d >= 1024): gradients near both ends of fp32's range, and gradients whose rows and
columns differ by more than the operands' own range.  Against the exact transform and the exact momentum in 64 bits on the device."""
import numpy as np
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _orthogonal(d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.linalg.qr(torch.randn((d, d), generator=g, device="cuda", dtype=torch.float64))[0].float().contiguous()


def _skew(R, G):
    P = G.double() @ R.double().T.contiguous()
    return 0.5 * (P - P.T)


def _rate(S, size):  # lr with lr ||S|| about `size` (power iteration)
    x = torch.ones((len(S), 1), device="cuda", dtype=torch.float64)
    for _ in range(60):
        x = S @ x
        x = x / x.norm()
    return float(np.float32(size / (S @ x).norm().item()))


def _momentum(R, G):
    """M after one step from a momentum of zero, and its exact value: S R with S from (1 - beta1) G, rounded to fp32 as the step does."""
    M, v, info = torch.zeros_like(R), torch.ones(1, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    kt.kt_cayley_adam_step(R.clone(), G, M, v, 1, 1e-3, info=info)
    M1 = G * float(np.float32(1) - np.float32(0.9))
    return M.double(), _skew(R, M1) @ R.double()


@pytest.mark.parametrize("gain", [1e-36, 1e-30, 1e30, 1e35])
@pytest.mark.parametrize("d", [1152, 2048])
def test_gradients_at_the_ends_of_the_range(d, gain):
    R = _orthogonal(d, d)
    g = torch.Generator(device="cuda").manual_seed(1)
    G = torch.randn((d, d), generator=g, device="cuda") * gain
    S = _skew(R, G)
    lr = _rate(S, 0.1)
    eye = torch.eye(d, device="cuda", dtype=torch.float64)
    want = torch.linalg.solve(eye + lr * S, R.double() - lr * S @ R.double())
    new, info = R.clone(), torch.zeros(1, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(new, G, lr, info=info)
    assert info.item() >= 1
    # the iteration ends within 0.75e-7 of its limit (a quarter of 3e-7), entry by entry; R and the last product round at 2^-24 of an entry
    # of at most 0.2 on top
    assert (new.double() - want).abs().max().item() <= 1.5e-7
    M, exact = _momentum(R, G)
    # two products of d terms in fp32: sqrt(d) 2^-24 of the norm each in the worst case, heads and tails 2^-23 an operand
    assert ((M - exact).norm() / exact.norm()).item() <= (2 * d ** 0.5 + 8) * 2.0 ** -24


@pytest.mark.parametrize("d", [1024, 1664])
def test_rows_and_columns_of_different_size(d):
    g = torch.Generator(device="cuda").manual_seed(d)
    rows, cols = (torch.exp2(-24 * torch.rand(d, generator=g, device="cuda")) for _ in range(2))
    G = torch.randn((d, d), generator=g, device="cuda") * rows[:, None] * cols[None]
    # a rotation that mixes the rows: as close as fp32 products are
    R = _orthogonal(d, d)
    M, exact = _momentum(R, G)
    assert ((M - exact).norm() / exact.norm()).item() <= (2 * d ** 0.5 + 8) * 2.0 ** -24
    # R = I keeps them apart: 2^-22 of the entries S is the difference of and of S (two operands each), or 2^-39 of the largest of them where
    # that is more (a head and tail of fp16 end 2^-40 below the largest magnitude of the operand, up to its leading bit)
    M, exact = _momentum(torch.eye(d, device="cuda"), G)
    P = 0.1 * (G.abs() + G.abs().T).double()
    bound = 2.0 ** -22 * (exact.abs() + P) + 2.0 ** -38 * P.max()
    assert ((M - exact).abs() / bound).max().item() <= 1.0
