"""fp32 products that read R and W as they lie (K as the row index of the tile) against a 64-bit product: edges of the 64 and
128 tiles on both sides, wide leading dimensions, and the copies that unaligned rows and a result over an operand still take."""
import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _matrix(rows, cols, ld, seed, offset=0):
    g = torch.Generator().manual_seed(seed)
    full = torch.randn(rows * ld + offset, generator=g, dtype=torch.float32).cuda()
    return full[offset:].as_strided((rows, cols), (ld, 1))


def _bound(a, b):
    # each sum of K products errs by at most K 2^-24 |a| |b| (and one rounding); in practice by sqrt(K)
    return (a.shape[1] * 2.0 ** -24) * (a.abs() @ b.abs()) + 1e-30


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("k,d,pad,offset", [(4, 128, 0, 0), (60, 128, 4, 0), (68, 256, 0, 0), (132, 384, 8, 0), (1000, 1024, 0, 0),
                                            (2052, 2048, 4, 0), (132, 256, 4, 1), (4, 128, 0, 3)])
def test_fuse_reads_the_operands_in_place(side, k, d, pad, offset):
    shape = (k, d) if side == 0 else (d, k)
    W = _matrix(*shape, shape[1] + pad, 1, offset if side == 1 else 0)
    R = _matrix(d, d, d + pad, 2, offset)
    out = torch.full(shape, float("nan"), device="cuda")
    kt.kt_fuse_rotation(W, R, side, out=out)
    A, B = (W.double(), R.double()) if side == 0 else (R.double().T.contiguous(), W.double())
    assert ((out.double() - A @ B).abs() <= _bound(A, B)).all()


@pytest.mark.parametrize("side", [0, 1])
def test_fuse_over_its_own_operand(side):
    d = 256
    W, R = _matrix(d, d, d, 3), _matrix(d, d, d, 4)
    want = kt.kt_fuse_rotation(W, R, side)
    over = R.clone()
    kt.kt_fuse_rotation(W, over, side, out=over)
    assert torch.equal(over, want)
    if side == 1:
        over = W.clone()
        kt.kt_fuse_rotation(over, R, side, out=over)
        assert torch.equal(over, want)


@pytest.mark.parametrize("batch,n,d", [(1, 1, 128), (2, 65, 256), (1, 130, 384), (1, 4100, 1024)])
def test_rotated_rows_fp32(batch, n, d):
    X = torch.stack([_matrix(n, d, d, 10 + b) for b in range(batch)])
    R = torch.stack([_matrix(d, d, d, 20 + b) for b in range(batch)]) / d ** 0.5
    Y = torch.empty((batch, n, d), device="cuda")
    kt.kt_rotate_quant_metrics(X, R, Y=Y)
    for b in range(batch):
        A, B = X[b].double(), R[b].double()
        assert ((Y[b].double() - A @ B).abs() <= _bound(A, B)).all()
    scales, codes = torch.empty((batch, n), device="cuda"), torch.empty((batch, n, d), dtype=torch.int8, device="cuda")
    kt.kt_rotate_fakequant_int4(X, R, scales_out=scales, codes=codes)
    given = torch.empty_like(codes)
    kt.kt_rotate_fakequant_int4(X, R, scales_in=scales, codes=given)
    amax = torch.empty_like(scales)
    kt.kt_rotate_fakequant_int4(X, R, scales_out=amax)
    # one tile's sums are in another order than the other's: a value on a rounding boundary may go either way
    assert (codes != given).float().mean() <= 1e-4
    torch.testing.assert_close(amax, scales, rtol=1e-5, atol=0)
    torch.testing.assert_close(scales, Y.abs().amax(2) / 7, rtol=1e-5, atol=0)


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("k,d", [(4, 256), (36, 384), (132, 512), (260, 128), (508, 1024), (516, 1024), (128, 4096)])
def test_few_tiles(side, k, d):
    """32 x 32 tiles with K shared by four waves: one to 32 steps a wave, ragged edges, either side of two tiles a CU."""
    W = _matrix(*((k, d) if side == 0 else (d, k)), d if side == 0 else k, 7)
    R = _matrix(d, d, d, 8)
    out = kt.kt_fuse_rotation(W, R, side)
    A, B = (W.double(), R.double()) if side == 0 else (R.double().T.contiguous(), W.double())
    assert ((out.double() - A @ B).abs() <= _bound(A, B)).all()


@pytest.mark.parametrize("batch,n,d,pad", [(1, 1, 128, 0), (2, 127, 256, 4), (1, 129, 640, 0), (1, 5000, 384, 8), (2, 300, 1152, 0),
                                           (1, 260, 4224, 0), (1, 70, 8320, 0)])
@pytest.mark.parametrize("unaligned", [False, True])
def test_row_loss_and_gradient_fp32(batch, n, d, pad, unaligned):
    """Rows of every register form (up to 1024, 4096, 8192 values and beyond), padding of the gradient product, wide rows of X, and R
    that has to be copied."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = (torch.randn((batch, n, d + pad), generator=g, device="cuda") + 0.3)[:, :, :d]
    ldr = d + 1 if unaligned and batch == 1 else d
    R = torch.randn((batch, d, ldr), generator=g, device="cuda")[:, :, :d] * d ** -0.5
    dR, kurt = torch.full((batch, d, d), float("nan"), device="cuda"), torch.empty((batch, n), device="cuda")
    loss = kt.kt_kurtosis_loss_grad(X, R, row_kurt=kurt, dR=dR)
    only = kt.kt_kurtosis_loss_grad(X, R)
    assert torch.equal(loss, only)
    for b in range(batch):
        x = X[b].double()
        y = x @ R[b].double()
        c = y - y.mean(1, keepdim=True)
        m2, m3, m4 = ((c ** k).mean(1, keepdim=True) for k in (2, 3, 4))
        kappa = m4 / m2 ** 2
        G = x.T.contiguous() @ (4.0 / y.numel() / m2 ** 2 * (c ** 3 - m3 - kappa * m2 * c))
        # y errs by about sqrt(d) 2^-24 of its size, a kurtosis by four times that, dR by sums of n terms on top
        assert ((kurt[b].double() - kappa[:, 0]).abs() <= 1e-5 * kappa[:, 0]).all()
        assert abs(loss[b].double() - kappa.mean()) <= 1e-5 * kappa.mean()
        assert (dR[b].double() - G).norm() <= 1e-5 * G.norm()


@pytest.mark.parametrize("batch,n,d,ldr,offset", [(2, 130, 256, 260, 0), (3, 33, 384, 392, 4), (1, 300, 640, 1024, 8), (2, 700, 512, 516, 0), (2, 20, 1152, 1156, 4),
                                                  (1, 40000, 128, 136, 0), (2, 9000, 256, 260, 4)])
def test_wide_aligned_rows_of_rotation(batch, n, d, ldr, offset):
    """R read in place with rows wider than d, one and several problems (d ldr apart): the same kernels and bits as with rows of d; NaN between
    the rows.  The last two sizes are past the line where the loss alone takes its row sums in the forward product."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn((batch, n, d), generator=g, device="cuda") + 0.3
    R = torch.randn((batch, d, d), generator=g, device="cuda") * d ** -0.5
    wide = torch.full((batch * d * ldr + offset,), float("nan"), device="cuda")[offset:].view(batch, d, ldr)[:, :, :d]
    wide.copy_(R)
    out = []
    for r in (R, wide):
        dR, kurt, pooled, kappa = (torch.empty(s, device="cuda") for s in ((batch, d, d), (batch, n), (batch, d, d), (batch,)))
        only = torch.empty_like(kurt)
        loss = kt.kt_kurtosis_loss_grad(X, r, row_kurt=kurt, dR=dR)
        alone = kt.kt_kurtosis_loss_grad(X, r, row_kurt=only)
        ploss = kt.kt_pooled_kurtosis_loss_grad(X, r, kappa=kappa, dR=pooled)
        palone = kt.kt_pooled_kurtosis_loss_grad(X, r)
        scales, err, codes = torch.empty((batch, n), device="cuda"), torch.empty((batch, n, 2), device="cuda"), torch.empty((batch, n, d), dtype=torch.int8, device="cuda")
        kt.kt_rotate_fakequant_int4(X, r, scales_out=scales, codes=codes, err=err)
        given = torch.empty_like(codes)
        kt.kt_rotate_fakequant_int4(X, r, scales_in=scales, codes=given)
        Y, thr = torch.empty_like(X), torch.empty((batch, n), device="cuda")
        kt.kt_rotate_quant_metrics(X, r, Y=Y, threshold=thr)
        out.append((loss, kurt, dR, alone, only, ploss, kappa, pooled, palone, scales, err, codes, given, Y, thr))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    for b in range(batch):
        A, B = X[b].double(), R[b].double()
        assert ((out[1][13][b].double() - A @ B).abs() <= _bound(A, B)).all()
