"""The launch whose tiles exchange the statistics of their token rows, with 256 x 256 tiles: one and two rounds of row blocks, ragged tokens, several
problems, d % 256 = 128 (the last tile half empty) and 0; and, both tile sizes, on a stream with so few CUs that tiles wait in vain, are
put on a list and made again.  Calls that take other launches would pass as well, so each looks whether it was this one."""
import ctypes

import pytest
import torch

import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu

LOSS = [(1, 7000, 1408), (1, 16001, 1408), (2, 3501, 1920), (1, 20001, 512), (1, 3001, 4096)]
QUANT = [(1, 7000, 1920), (2, 3500, 1920), (1, 16700, 1408), (1, 11500, 1024)]


def _problem(batch, n, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn((batch, n, d), generator=g, device="cuda")
    X[:, :, :3] *= 30.0
    X[:, ::7] = X[:, ::7] ** 3 / 4
    R = torch.stack([torch.linalg.qr(torch.randn((d, d), generator=g, device="cuda"))[0] for _ in range(batch)]).contiguous()
    return X.bfloat16(), R


def _loss_in_64_bits(X, R):
    X, R = X.double(), R.bfloat16().double()
    Y = X @ R
    c = Y - Y.mean(1, keepdim=True)
    m2, m3, m4 = ((c ** k).mean(1, keepdim=True) for k in (2, 3, 4))
    kappa = m4 / m2 ** 2
    G = 4.0 / (Y.shape[0] * Y.shape[1] * m2 ** 2) * (c ** 3 - m3 - kappa * m2 * c)
    return kappa[:, 0], X.T @ G


def _launches_of(kernel_id, call):
    kt.kt_profile_enable(8)
    try:
        kt.kt_profile_reset()
        out = call()
        return out, kt.kt_profile_read(kernel_id)[1]
    finally:
        kt.kt_profile_enable(0)


@pytest.mark.parametrize("batch,n,d", LOSS)
def test_loss_and_gradient(batch, n, d):
    X, R = _problem(batch, n, d, seed=n + d)
    dR, rk = torch.full((batch, d, d), float("nan"), device="cuda"), torch.full((batch, n), float("nan"), device="cuda")
    loss, of_its_own = _launches_of(1, lambda: kt.kt_kurtosis_loss_grad(X, R, dR=dR, row_kurt=rk))
    assert of_its_own == 0  # dL/dY left the forward product
    for b in range(batch):
        kappa, want = _loss_in_64_bits(X[b], R[b])
        # y is off by a few 2^-24 of its row, its fourth moment by the like
        assert torch.allclose(rk[b].double(), kappa, rtol=1e-4, atol=0)
        assert abs(loss[b].item() - kappa.mean().item()) <= 1e-5 * kappa.mean().item()
        assert (dR[b].double() - want).norm() <= 6e-3 * want.norm()  # dL/dY is rounded to bf16 (2^-9 an entry)


def _quantise(X, R, ws=None):
    batch, n, d = X.shape
    codes = torch.full((batch, n, d), 99, dtype=torch.int8, device="cuda")
    scales, err = torch.full((batch, n), float("nan"), device="cuda"), torch.full((batch, n, 2), float("nan"), device="cuda")
    kt.kt_rotate_fakequant_int4(X, R, clip_ratio=0.9, scales_out=scales, codes=codes, err=err, workspace=ws)
    return codes, scales, err


def _unstaged(X, R):
    """_quantise, and that the rotated rows (4 n d bytes) have not been in the workspace."""
    ws = kt.Workspace("cuda")
    ws.get(kt.kt_workspace_bytes(kt.KT_OP_FAKEQUANT, *X.shape, kt.KT_BF16)).fill_(0x5a)
    out = _quantise(X, R, ws)
    assert int((ws.buf != 0x5a).sum()) < 2 * X.numel() + 2 * R.numel()
    return out


@pytest.mark.parametrize("batch,n,d", QUANT)
def test_fakequant(batch, n, d):
    X, R = _problem(batch, n, d, seed=n + d)
    codes, scales, err = _unstaged(X, R)
    for b in range(batch):
        y = X[b].double() @ R[b].bfloat16().double()
        s = scales[b].double()[:, None]
        # fp32 sums of d products: a few ulp of the row's magnitude
        assert torch.allclose(s, 0.9 * y.abs().amax(1, keepdim=True) / 7, rtol=2e-5, atol=0)
        v, c = y / s, codes[b].double()
        away = (v - (v.floor() + 0.5)).abs() > 1e-3  # from a rounding boundary
        assert torch.equal(c[away], v.round().clamp(-7, 7)[away]) and bool((c.abs() <= 7).all())
        assert torch.allclose(err[b, :, 0].double(), ((y - c * s) ** 2).sum(1), rtol=1e-4, atol=0)
        assert torch.allclose(err[b, :, 1].double(), (y * y).sum(1), rtol=1e-4, atol=0)


def _few_cu_stream(cus):
    """A stream that may use `cus` compute units (None where the runtime has no such streams)."""
    hip = ctypes.CDLL("libamdhip64.so")
    words = (ctypes.c_uint32 * 8)(*([(1 << cus) - 1] + [0] * 7))
    st = ctypes.c_void_p()
    if not hasattr(hip, "hipExtStreamCreateWithCUMask") or hip.hipExtStreamCreateWithCUMask(ctypes.byref(st), 8, words) != 0:
        return None
    return torch.cuda.ExternalStream(st.value)


def _on_few_cus(call):
    st = _few_cu_stream(8)
    if st is None:
        pytest.skip("no streams with a CU mask")
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        out = call()
        st.synchronize()
    return out


@pytest.mark.parametrize("n,d", [(3000, 4096), (5000, 640)])  # tiles of 256, of 128
def test_fakequant_on_few_cus(n, d):
    X, R = _problem(1, n, d, seed=11)
    want = _unstaged(X, R)
    got = _on_few_cus(lambda: _quantise(X, R))
    for a, b in zip(want, got):
        assert torch.equal(a, b)


def test_large_loss_tiles_on_few_cus():
    X, R = _problem(1, 3000, 4096, seed=12)

    def call():
        dR, rk = torch.full((1, 4096, 4096), float("nan"), device="cuda"), torch.full((1, 3000), float("nan"), device="cuda")
        return kt.kt_kurtosis_loss_grad(X, R, dR=dR, row_kurt=rk), rk, dR

    for a, b in zip(call(), _on_few_cus(call)):
        assert torch.equal(a, b)
