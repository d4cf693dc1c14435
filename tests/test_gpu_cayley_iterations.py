"""Retractions of many iterations: the first 3, 6, 8, 16 or all as launches of their own, the later ones inside one launch (release or stores past the L2), on tile grids on either
side of each rule, one and several problems; Cayley Adam with both forms of the products and with control words that do not fit
their first place (d = 5760).  Against the exact transform in 64 bits on the device."""
import numpy as np
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _orthogonal(d, g):
    return torch.linalg.qr(torch.randn((d, d), generator=g, device="cuda", dtype=torch.float64))[0].float()


def _skew(R, G):
    P = G.double() @ R.double().T.contiguous()
    return 0.5 * (P - P.T)


def _transform(R, A):
    eye = torch.eye(len(R), device="cuda", dtype=torch.float64)
    return torch.linalg.solve(eye + A, R.double() - A @ R.double())


# (problems, d, (lr / 2) ||A||, least iterations)
@pytest.mark.parametrize("batch,d,size,least", [(1, 256, 0.3, 9), (8, 256, 0.3, 9), (32, 256, 0.3, 9), (130, 256, 0.3, 9), (4, 512, 0.5, 18), (1, 640, 0.5, 17), (1, 768, 0.3, 9),
                                                (2, 896, 0.5, 18), (1, 1024, 0.3, 9), (1, 1152, 0.3, 9), (1, 1408, 0.5, 17), (2, 1024, 0.3, 9),
                                                (1, 2048, 0.3, 9), (1, 2432, 0.3, 9)])
def test_many_iterations(batch, d, size, least):
    g = torch.Generator(device="cuda").manual_seed(batch + d)
    R = torch.stack([_orthogonal(d, g) for _ in range(batch)])
    G = torch.randn((batch, d, d), generator=g, device="cuda")
    for b in range(batch):  # one lr for all problems
        S = _skew(R[b], G[b])
        x = torch.ones((d, 1), device="cuda", dtype=torch.float64)
        for _ in range(60):
            x = S @ x
            x = x / x.norm()
        G[b] *= size * (b + 2) / (batch + 1) / (S @ x).norm().item()  # the last problem `size`, the others less
    lr = 1.0
    new, info = R.clone(), torch.zeros(batch, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(new, G, lr, info=info)
    assert info.min().item() >= 1 and info.max().item() >= least
    for b in {0, batch - 1}:
        # the iteration ends within a quarter of 3e-7 of its limit; its products and R itself round at 2^-24 of an entry below 0.5
        assert (new[b].double() - _transform(R[b], lr * _skew(R[b], G[b]))).abs().max().item() <= 3e-7


@pytest.mark.parametrize("d,small_workspace", [(640, False), (1152, False), (1152, True), (1664, False), (2176, True), (5760, False)])
def test_adam_many_iterations(d, small_workspace):
    """A gradient of rank one: half of 1 = 2 q goes into each of two singular values, which takes a dozen iterations."""
    g = torch.Generator(device="cuda").manual_seed(d)
    R = _orthogonal(d, g).contiguous()
    G = torch.randn((d, 1), generator=g, device="cuda") @ torch.randn((1, d), generator=g, device="cuda")
    full = kt.kt_workspace_bytes(kt.KT_OP_CAYLEY, 1, 0, d, kt.KT_F32)
    size = full - (10 * d * d if small_workspace else 0)  # five d x d matrices of fp32 instead of three and three split ones

    class Exactly:
        def get(self, need):
            return torch.empty(size + 256, dtype=torch.uint8, device="cuda")[:size]

    new, M, v = R.clone(), torch.zeros_like(R), torch.ones(1, device="cuda")
    info, scalars = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.empty((1, 3), device="cuda")
    kt.kt_cayley_adam_step(new, G, M, v, 1, 1e3, info=info, scalars=scalars, workspace=Exactly())
    assert info.item() >= 9
    M1 = G * float(np.float32(1) - np.float32(0.9))
    S = _skew(R, M1)
    r, a, w = scalars[0].double().tolist()
    assert abs(w * r / S.norm().item() - 1) <= 1e-5 and abs(a * (w + 1e-8) - 1) <= 1e-5
    exact = S @ R.double()
    # sqrt(d) 2^-24 of the norm for each of two products of d terms in fp32, and the heads and tails
    assert ((M.double() - exact).norm() / exact.norm()).item() <= (2 * d ** 0.5 + 8) * 2.0 ** -24
    want = _transform(R, 0.5 * a / r * S)
    # as above, and the factor a / (2 r) in fp32
    assert (new.double() - want).abs().max().item() <= 3e-7 + 2.0 ** -22 * (want - R.double()).abs().max().item()
