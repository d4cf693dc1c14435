"""Retractions whose products run on fp16 heads and tails (d >= 1024): every tile with full and half-empty ends, gradients of extreme sizes
(each operand is scaled by a power of two from its largest magnitude), non-finite ones, and the workspace that only holds
the fp32 form.  Against the exact Cayley transform in 64 bits on the device."""
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _problem(d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    R = torch.linalg.qr(torch.randn((d, d), generator=g, device="cuda", dtype=torch.float64))[0].float().contiguous()
    G = torch.randn((d, d), generator=g, device="cuda")
    G[:, ::61] *= 100.0
    return R, G


def _exact(R, G, lr):
    K = G.double() @ R.double().T.contiguous()
    a = 0.5 * lr * (K - K.T)
    eye = torch.eye(len(R), device="cuda", dtype=torch.float64)
    return torch.linalg.solve(eye + a, R.double() - a @ R.double())


def _lr(R, G, size):  # (lr / 2) ||A|| about `size`
    K = G.double() @ R.double().T.contiguous()
    return 2.0 * size / torch.linalg.matrix_norm(K - K.T, 2).item()


@pytest.mark.parametrize("d,size,gain", [(1024, 0.05, 1.0), (1152, 0.3, 1e-20), (1664, 0.05, 1e15), (2176, 0.01, 1.0), (3200, 0.05, 1.0)])
def test_step(d, size, gain):
    R, G = _problem(d, d)
    lr = _lr(R, G, size) / gain
    G = G * gain
    want = _exact(R, G, lr)
    new, info, err = R.clone(), torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")
    kt.kt_cayley_step(new, G, lr, info=info, ortho_err=err)
    assert info.item() >= 1 and err.item() < 1e-6
    # R is stored in fp32: 2^-24 of its entries' norm, and about as much again for each of the last products
    assert (new.double() - want).norm() <= 4e-7 * d ** 0.5


def test_several_problems():
    R, G = (torch.stack(t) for t in zip(*(_problem(1152, s) for s in (1, 2, 3))))
    G = (G * torch.tensor([1.0, 1e-6, 1e6], device="cuda").view(3, 1, 1)).contiguous()
    for b in range(3):
        G[b] *= _lr(R[b], G[b], 0.1) / 1e-2
    new = R.clone()
    kt.kt_cayley_step(new, G, 1e-2)
    for b in range(3):
        one = R[b].clone()
        kt.kt_cayley_step(one, G[b], 1e-2)
        assert (new[b].double() - _exact(R[b], G[b], 1e-2)).norm() <= 4e-7 * 1152 ** 0.5
        assert (one - new[b]).norm() <= 4e-7 * 1152 ** 0.5


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_non_finite_gradient_is_rejected(bad):
    R, G = _problem(1152, 5)
    G[7, 9] = bad
    new, info = R.clone(), torch.zeros(1, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(new, G, 1e-3, info=info)
    assert info.item() < 1 and torch.equal(new, R)


def test_smaller_workspace_takes_the_fp32_products():
    d = 1152
    R, G = _problem(d, 6)
    lr = _lr(R, G, 0.1)
    full = kt.kt_workspace_bytes(kt.KT_OP_CAYLEY, 1, 0, d, kt.KT_F32)
    small = full - 10 * d * d  # five d x d matrices of fp32 instead of three and three split ones

    class Exactly:
        def get(self, need):
            return torch.empty(small + 256, dtype=torch.uint8, device="cuda")[:small]

    new, info = R.clone(), torch.zeros(1, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(new, G, lr, info=info, workspace=Exactly())
    assert info.item() >= 1 and (new.double() - _exact(R, G, lr)).norm() <= 4e-7 * d ** 0.5
