"""Calls that leave most of the chip without a tile take other kernels than large ones: a handful of tokens straight from
R, small tiles for few outputs.  Each at the edges of its range, element by element against a 64-bit product; the bound is that of
an fp32 sum of d products in any order, d 2^-24 sum |x| |r| (the products of bf16 values are exact), doubled for the
partial sums."""
import numpy as np
import pytest
import torch

import ktgen
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _problem(batch, n, d, xdt, rdt, ld_pad, seed):
    X = torch.stack([ktgen.make_x(n, d, seed=seed + b, outlier_cols=3, outlier_scale=40.0, dtype=xdt) for b in range(batch)])
    R = torch.stack([ktgen.random_orthogonal(d, seed=seed + 10 + b) for b in range(batch)])
    if rdt == "bf16":
        R = R.to(torch.bfloat16)
    wide = torch.full((batch, d, d + ld_pad), 7.0, dtype=R.dtype)
    wide[:, :, :d] = R
    return X.cuda(), wide.cuda()[:, :, :d], R


@pytest.mark.parametrize("batch,n,d,xdt,rdt,ld_pad", [
    (1, 1, 256, "bf16", "f32", 0), (1, 16, 1152, "bf16", "f32", 4), (2, 17, 384, "bf16", "f32", 0),
    (1, 32, 128, "bf16", "bf16", 8), (3, 33, 640, "bf16", "bf16", 0), (1, 64, 2048, "bf16", "f32", 0),
    (1, 5, 512, "bf16", "f32", 1),      # rows of R not 16-byte aligned: general path
    (1, 65, 2048, "bf16", "f32", 0), (1, 700, 896, "bf16", "f32", 0), (1, 130, 384, "f32", "f32", 0),
    # 256 x 128 tiles, ragged rows: 132 and 432 (one round, two nearly full ones); 128 x 128 for 258 and 513
    (44, 200, 384, "bf16", "f32", 0), (36, 1000, 384, "bf16", "f32", 0), (86, 130, 384, "bf16", "f32", 0), (57, 600, 384, "bf16", "f32", 0),
])
def test_rotated_rows(batch, n, d, xdt, rdt, ld_pad):
    X, R, Rh = _problem(batch, n, d, xdt, rdt, ld_pad, 3 * n + d)
    Y = torch.full((batch, n, d), float("nan"), device="cuda")
    thr = torch.empty((batch, n), device="cuda")
    kt.kt_rotate_quant_metrics(X, R, quantile=1.0, Y=Y, threshold=thr)
    scales = torch.empty((batch, n), device="cuda")
    codes = torch.empty((batch, n, d), dtype=torch.int8, device="cuda")
    err = torch.empty((batch, n, 2), device="cuda")
    kt.kt_rotate_fakequant_int4(X, R, scales_out=scales, codes=codes, err=err)
    torch.cuda.synchronize()
    for b in range(batch):
        x = ktgen.to_f64(X[b])
        r = ktgen.to_f64(ktgen.bf16_round(Rh[b]) if xdt == "bf16" else Rh[b])
        ref, bound = x @ r, 2.0 * d * 2.0 ** -24 * (np.abs(x) @ np.abs(r))
        y = Y[b].cpu().double().numpy()
        assert np.all(np.abs(y - ref) <= bound)
        assert np.array_equal(thr[b].cpu().numpy(), np.abs(y).max(1).astype(np.float32))
        s = scales[b].cpu().numpy()
        assert np.all(np.abs(s - np.abs(ref).max(1) / 7) <= (bound.max(1) + 1e-6 * np.abs(ref).max(1)) / 7)
        # codes from the library's own scale: off by rounding only where the value sits within the bound of a boundary
        v = ref / s[:, None].astype(np.float64)
        q = codes[b].cpu().numpy()
        off = np.abs(q - np.clip(v, -7, 7)) - 0.5
        assert np.all(off <= bound / s[:, None] + 1e-5)
        e = ((ref - q * s[:, None].astype(np.float64)) ** 2).sum(1)
        assert np.allclose(err[b, :, 0].cpu().numpy(), e, rtol=1e-4) and np.allclose(err[b, :, 1].cpu().numpy(), (ref ** 2).sum(1), rtol=1e-4)


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("k,d", [(4, 128), (132, 256), (1000, 384), (2052, 2048), (5632, 2048)])
def test_fused_weights_small_and_large_tiles(side, k, d):
    """The number of 128 x 128 tiles decides the tile: 1 to 24 and, a little over one round of CUs, 272 and 704, all small
    (sizes for the large one: test_gpu_large_fp32_tiles.py)."""
    g = torch.Generator().manual_seed(k + d)
    W = torch.randn((k, d) if side == 0 else (d, k), generator=g)
    R = ktgen.random_orthogonal(d, seed=k)
    out = kt.kt_fuse_rotation(W.cuda(), R.cuda(), side)
    torch.cuda.synchronize()
    w, r = W.double().numpy(), R.double().numpy()
    ref = w @ r if side == 0 else r.T @ w
    size = np.abs(w) @ np.abs(r) if side == 0 else np.abs(r).T @ np.abs(w)
    assert np.all(np.abs(out.cpu().double().numpy() - ref) <= d * 2.0 ** -23 * size)


@pytest.mark.parametrize("batch,n", [
    (1, 1), (1, 15), (3, 64), (256, 64), (255, 17), (1, 16384),      # one tile per wave
    (256, 65), (128, 256), (129, 100), (1, 16385), (129, 129),       # two
    (257, 64), (600, 33), (40, 1000), (513, 300),                    # two workgroups per CU, several tiles per wave, rounds
])
def test_heads_of_128_in_every_launch_shape(batch, n):
    """The d = 128 fake-quant, all tokens of all problems, with its own scales and with given ones (its own again: the same
    arithmetic, so the same codes)."""
    d = 128
    X, R, Rh = _problem(1, batch * n, d, "bf16", "f32", 0, batch + n)
    X = X.view(batch, n, d)
    Rd = torch.stack([torch.roll(R[0], b, 1) for b in range(batch)])   # a rotation of its own for every problem
    scales, codes, err = (torch.full((batch, n), -1.0, device="cuda"), torch.full((batch + 1, n, d), 99, dtype=torch.int8, device="cuda"),
                          torch.full((batch, n, 2), -1.0, device="cuda"))
    kt.kt_rotate_fakequant_int4(X, Rd, scales_out=scales, codes=codes[:batch], err=err)
    again = torch.full_like(codes, 99)
    kt.kt_rotate_fakequant_int4(X, Rd, scales_in=scales, codes=again[:batch])
    torch.cuda.synchronize()
    assert torch.equal(codes, again) and bool((codes[batch] == 99).all())
    r = ktgen.to_f64(ktgen.bf16_round(Rh[0]))
    x = ktgen.to_f64(X.reshape(batch * n, d))
    shift = (np.arange(d)[None, :] - np.repeat(np.arange(batch), n)[:, None]) % d
    ref = np.take_along_axis(x @ r, shift, 1)
    bound = np.take_along_axis(2.0 * d * 2.0 ** -24 * (np.abs(x) @ np.abs(r)), shift, 1)
    s = scales.cpu().double().numpy().reshape(-1)
    assert np.all(np.abs(s - np.abs(ref).max(1) / 7) <= (bound.max(1) + 1e-6 * np.abs(ref).max(1)) / 7)
    q = codes[:batch].cpu().numpy().reshape(-1, d)
    assert np.all(np.abs(q - np.clip(ref / s[:, None], -7, 7)) - 0.5 <= bound / s[:, None] + 1e-5)
    e = err.cpu().numpy().reshape(-1, 2)
    assert np.allclose(e[:, 0], ((ref - q * s[:, None]) ** 2).sum(1), rtol=1e-4) and np.allclose(e[:, 1], (ref ** 2).sum(1), rtol=1e-4)


@pytest.mark.parametrize("batch,n,d,rdt", [(1, 1, 4096, "f32"), (1, 16, 4096, "f32"), (2, 33, 1152, "bf16"), (1, 64, 2048, "f32"), (1, 65, 2048, "f32")])
def test_own_scales_handed_back(batch, n, d, rdt):
    """With given scales y comes from the GEMM, without them and up to 64 tokens from the few-token kernel, whose sums have
    another order: a code may differ where y / s lies that close to a rounding boundary, and by one only."""
    X, R, Rh = _problem(batch, n, d, "bf16", rdt, 0, n + d)
    scales, codes, again = (torch.empty((batch, n), device="cuda"), torch.empty((batch, n, d), dtype=torch.int8, device="cuda"),
                            torch.empty((batch, n, d), dtype=torch.int8, device="cuda"))
    kt.kt_rotate_fakequant_int4(X, R, scales_out=scales, codes=codes)
    kt.kt_rotate_fakequant_int4(X, R, scales_in=scales, codes=again)
    torch.cuda.synchronize()
    if n > 64:
        assert torch.equal(codes, again)
    for b in range(batch):
        x, r, s = ktgen.to_f64(X[b]), ktgen.to_f64(ktgen.bf16_round(Rh[b])), scales[b].cpu().double().numpy()[:, None]
        v, slack = x @ r / s, 2.0 * d * 2.0 ** -24 * (np.abs(x) @ np.abs(r)) / s + 1e-5
        diff = codes[b].cpu().numpy().astype(int) - again[b].cpu().numpy()
        assert np.abs(diff).max() <= 1
        assert np.all(np.abs(np.abs(v - np.floor(v)) - 0.5)[diff != 0] <= slack[diff != 0])


@pytest.mark.parametrize("n,more,d", [(65, 4000, 1408), (700, 3000, 1408), (129, 9000, 2048), (1500, 5000, 2048), (1001, 4100, 2688), (400, 9000, 4096), (1000, 4100, 4096)])
def test_a_token_has_the_bits_it_has_in_a_larger_call(n, more, d):
    """From 65 tokens on y, and with it the scale and the codes, does not depend on how many other tokens there are, nor on whose scales are
    used: every sum over the d products has one order, whatever the tiles."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn((1, more, d), generator=g, device="cuda").bfloat16()
    R = torch.linalg.qr(torch.randn((1, d, d), generator=g, device="cuda"))[0].contiguous()

    def rotated(m):
        Y, scales = torch.empty((1, m, d), device="cuda"), torch.empty((1, m), device="cuda")
        codes, given = torch.empty((1, m, d), dtype=torch.int8, device="cuda"), torch.empty((1, m, d), dtype=torch.int8, device="cuda")
        kt.kt_rotate_quant_metrics(X[:, :m], R, Y=Y)
        kt.kt_rotate_fakequant_int4(X[:, :m], R, scales_out=scales, codes=codes)
        kt.kt_rotate_fakequant_int4(X[:, :m], R, scales_in=scales, codes=given)
        return Y, scales, codes, given

    few, many = rotated(n), rotated(more)
    for a, b in zip(few, many):
        assert torch.equal(a, b[:, :n])
    assert torch.equal(few[2], few[3]) and torch.equal(many[2], many[3])
    assert torch.equal(few[1], few[0].abs().amax(2) / torch.full_like(few[1], 7.0))  # (by a number torch multiplies with its reciprocal)


@pytest.mark.parametrize("n,limit", [(16384, 4.6e-7), (8192, 3.2e-7)])
def test_fp32_gradient_keeps_its_precision_over_many_tokens(n, limit):
    """dR = X^T G sums over the tokens in fp32, in 16 ranges whatever the tile: the relative error of dR is 3.5e-7 and 2.5e-7
    for these inputs.  64 x 64 tiles with a quarter of the ranges, sums four times as long, came to 5.9e-7 and 3.9e-7; the
    limits lie half way."""
    d = 1024
    g = torch.Generator().manual_seed(n + 1)
    X = (torch.randn(n, d, generator=g) * torch.exp(torch.randn(d, generator=g))).cuda()
    R = ktgen.random_orthogonal(d, seed=d).cuda()
    dR = torch.empty((1, d, d), device="cuda")
    kt.kt_kurtosis_loss_grad(X[None], R[None], dR=dR)
    x = X.double()
    y = x @ R.double()
    c = y - y.mean(1, keepdim=True)
    m2, m3 = (c * c).mean(1, keepdim=True), (c ** 3).mean(1, keepdim=True)
    kappa = (c ** 4).mean(1, keepdim=True) / m2 ** 2
    ref = x.T.contiguous() @ (4.0 / (n * d) / m2 ** 2 * (c ** 3 - m3 - kappa * m2 * c))
    assert ((dR[0].double() - ref).norm() / ref.norm()).item() <= limit
