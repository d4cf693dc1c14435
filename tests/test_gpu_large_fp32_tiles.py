"""fp32 products with so many outputs that 128 x 128 tiles fill the CUs (fewer take 64 x 64): every entry point that has
them, with rows and columns that end inside a tile.  The batched calls repeat four problems, so that every problem is
checked: the first four against the oracle, the others against their twin, bit for bit."""
import numpy as np
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt
from parity_util import check_loss_grad, gpu_loss_grad, oracle_loss_grad, rel_fro

pytestmark = pytest.mark.gpu

D, BATCH, DISTINCT = 256, 128, 4


def _large(tiles):
    """The library's rule for 128 x 128 tiles: more than the 256 CUs, the last round of them nearly full."""
    rounds = -(-tiles // 256) * 256
    return tiles > 256 and 33 * tiles >= 32 * rounds


def _twins(t):
    return t.repeat(BATCH // DISTINCT, *[1] * (t.dim() - 1))


def _assert_twins(t):
    t = t.reshape(BATCH // DISTINCT, DISTINCT, -1)
    assert torch.equal(t, t[:1].expand_as(t))


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("k,d", [(4092, 2048), (16260, 512)])
def test_fused_weights(side, k, d):
    assert _large(-(-k // 128) * (d // 128))
    g = torch.Generator().manual_seed(k + d)
    W = torch.randn((k, d) if side == 0 else (d, k), generator=g)
    R = ktgen.random_orthogonal(d, seed=k)
    out = kt.kt_fuse_rotation(W.cuda(), R.cuda(), side)
    torch.cuda.synchronize()
    # 64-bit product of sampled rows and columns: each edge of the matrix and of a tile
    rows = np.unique(np.r_[0, 1, 127, 128, out.shape[0] - 129, out.shape[0] - 2, out.shape[0] - 1])
    w, r = W.double().numpy(), R.double().numpy()
    if side == 0:
        ref, size = w[rows] @ r, np.abs(w[rows]) @ np.abs(r)
    else:
        ref, size = r.T[rows] @ w, np.abs(r.T[rows]) @ np.abs(w)
    assert np.all(np.abs(out.cpu().double().numpy()[rows] - ref) <= d * 2.0 ** -23 * size)


def _rotations():
    return torch.stack([ktgen.random_orthogonal(D, seed=b) for b in range(DISTINCT)])


def test_cayley_step():
    assert _large((D // 128) ** 2 * BATCH)
    g = torch.Generator().manual_seed(1)
    R, G = _rotations(), torch.randn((DISTINCT, D, D), generator=g) * 3.0 / np.sqrt(D)
    Rd, oe, info = _twins(R).cuda(), torch.zeros(BATCH, device="cuda"), torch.zeros(BATCH, dtype=torch.int32, device="cuda")
    kt.kt_cayley_step(Rd, _twins(G).cuda(), 1e-2, ortho_err=oe, info=info)
    torch.cuda.synchronize()
    _assert_twins(Rd), _assert_twins(oe), _assert_twins(info)
    for b in range(DISTINCT):
        r0, rn = ktgen.to_f64(R[b]), Rd[b].cpu().double().numpy()
        assert rel_fro(rn - r0, oracle.cayley_step(r0, ktgen.to_f64(G[b]), 1e-2) - r0) <= 1e-4
        true = np.abs(rn.T @ rn - np.eye(D)).max()
        assert true < 1e-6 and abs(oe[b].item() - true) < 6e-7 and 1 <= info[b].item() <= 32


def test_cayley_adam_step():
    g = torch.Generator().manual_seed(2)
    R, G = _rotations(), torch.randn((DISTINCT, D, D), generator=g) * 5.0 / np.sqrt(D)
    M, v = 0.3 * torch.randn((DISTINCT, D, D), generator=g) / np.sqrt(D), torch.rand(DISTINCT, generator=g) + 0.5
    Rd, Md, vd = _twins(R).cuda(), _twins(M).cuda(), _twins(v).cuda()
    kt.kt_cayley_adam_step(Rd, _twins(G).cuda(), Md, vd, 2, 0.1)
    torch.cuda.synchronize()
    _assert_twins(Rd), _assert_twins(Md), _assert_twins(vd)
    f32 = lambda x: float(np.float32(x))  # noqa: E731  (the C interface takes fp32 hyper-parameters)
    for b in range(DISTINCT):
        o = oracle.cayley_adam_step(ktgen.to_f64(R[b]), ktgen.to_f64(G[b]), ktgen.to_f64(M[b]), float(v[b]), 2, f32(0.1),
                                    beta1=f32(0.9), beta2=f32(0.99), eps=f32(1e-8), q=0.5)
        r0 = ktgen.to_f64(R[b])
        assert rel_fro(Rd[b].cpu().double().numpy() - r0, o["R"] - r0) <= 1e-4
        assert rel_fro(Md[b].cpu().double().numpy(), o["M"]) <= 1e-4


def test_loss_grad():
    X = torch.stack([ktgen.make_x(203, D, seed=b, outlier_cols=3, outlier_scale=30.0, t_frac=0.05, dtype="f32") for b in range(DISTINCT)])
    R = _rotations()
    g = gpu_loss_grad(_twins(X), _twins(R))
    for key in ("loss", "row_kurt", "dR"):
        _assert_twins(torch.from_numpy(g[key]))
        g[key] = g[key][:DISTINCT]
    check_loss_grad(g, oracle_loss_grad(X, R), 1e-4)


def test_fake_quant_and_metrics():
    n = 130
    assert _large(-(-n // 128) * (D // 128) * BATCH)
    X = torch.stack([ktgen.make_x(n, D, seed=b, outlier_cols=3, outlier_scale=30.0, dtype="f32") for b in range(DISTINCT)])
    R = _rotations()
    Xd, Rd = _twins(X).cuda(), _twins(R).cuda()
    Y, scales = torch.empty((BATCH, n, D), device="cuda"), torch.empty((BATCH, n), device="cuda")
    codes = torch.empty((BATCH, n, D), dtype=torch.int8, device="cuda")
    kt.kt_rotate_quant_metrics(Xd, Rd, quantile=1.0, Y=Y)
    kt.kt_rotate_fakequant_int4(Xd, Rd, scales_out=scales, codes=codes)
    torch.cuda.synchronize()
    _assert_twins(Y), _assert_twins(scales), _assert_twins(codes)
    for b in range(DISTINCT):
        x, r, y = ktgen.to_f64(X[b]), ktgen.to_f64(R[b]), Y[b].cpu().double().numpy()
        assert np.all(np.abs(y - x @ r) <= D * 2.0 ** -23 * (np.abs(x) @ np.abs(r)))
        s = scales[b].cpu().numpy()
        assert np.array_equal(s, (np.abs(Y[b].cpu().numpy()).max(1) / np.float32(7)).astype(np.float32))
        q = np.clip(np.rint(Y[b].cpu().numpy() * (np.float32(1) / s)[:, None]), -7, 7)   # the definition, in fp32
        assert np.array_equal(codes[b].cpu().numpy(), q.astype(np.int8))
