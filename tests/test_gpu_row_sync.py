"""Loss + gradient and fake-quant where the tiles of a token row exchange its statistics inside the launch: the edges of the
128 and 256 token blocks and of the 256-feature tiles (d % 256 = 128: the last one half empty), fewer and more row blocks than
are in flight, several problems, and a stream with fewer CUs than a row has tiles, where tiles wait in vain and are made
again."""
import ctypes

import numpy as np
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu

# (batch, n, d): one row block and its edges, more row blocks than in flight (d = 384: 170 of 128 tokens; 256: 256 of 256), a ragged last one
LOSS = [(1, 64, 256), (1, 127, 384), (1, 129, 256), (2, 255, 640), (1, 257, 1152), (3, 700, 384), (1, 2500, 1408), (1, 23000, 384), (1, 66001, 256)]
QUANT = [(1, 12000, 256), (2, 6001, 384), (1, 23001, 640), (1, 10001, 1024), (1, 5800, 1920), (1, 66001, 256)]


def _problem(batch, n, d, seed):
    X = ktgen.make_x(n * batch, d, seed=seed, outlier_cols=3, outlier_scale=30.0, t_frac=0.05, dtype="bf16").reshape(batch, n, d)
    R = torch.stack([ktgen.random_orthogonal(d, seed=seed + 100 * b) for b in range(batch)])
    return X, R


@pytest.mark.parametrize("batch,n,d", LOSS)
def test_loss_and_gradient_against_oracle(batch, n, d):
    X, R = _problem(batch, n, d, seed=7)
    Xc, Rc = X.cuda(), R.cuda()
    dR = torch.full((batch, d, d), float("nan"), device="cuda")
    rk = torch.full((batch, n), float("nan"), device="cuda")
    loss = kt.kt_kurtosis_loss_grad(Xc, Rc, dR=dR, row_kurt=rk)
    only = kt.kt_kurtosis_loss_grad(Xc, Rc)  # no gradient: the row statistics are a launch of their own
    torch.cuda.synchronize()
    # two fp32 roundings of each partial, merged in fp64: 2^-23 of a moment
    assert torch.allclose(loss, only, rtol=1e-6, atol=0)
    for b in range(batch):
        o = oracle.loss_grad(ktgen.to_f64(X[b]), ktgen.to_f64(ktgen.bf16_round(R[b])))
        assert abs(loss[b].item() - o["loss"]) <= 1e-5 * abs(o["loss"])
        err = np.linalg.norm(dR[b].cpu().numpy().astype(np.float64) - o["dR"]) / np.linalg.norm(o["dR"])
        assert err <= 6e-3, err  # dL/dY is rounded to bf16 (2^-9 an entry)
    assert torch.isfinite(rk).all()
    assert torch.allclose(rk.double().mean(1), loss.double(), rtol=1e-5)


@pytest.mark.parametrize("batch,n,d", QUANT)
def test_fakequant_against_oracle(batch, n, d):
    X, R = _problem(batch, n, d, seed=8)
    sc = torch.full((batch, n), float("nan"), device="cuda")
    err = torch.full((batch, n, 2), float("nan"), device="cuda")
    codes = torch.full((batch, n, d), 99, dtype=torch.int8, device="cuda")
    kt.kt_rotate_fakequant_int4(X.cuda(), R.cuda(), clip_ratio=0.9, scales_out=sc, codes=codes, err=err)
    torch.cuda.synchronize()
    for b in range(batch):
        y = ktgen.to_f64(X[b]) @ ktgen.to_f64(ktgen.bf16_round(R[b]))
        s = sc[b].cpu().numpy().astype(np.float64)
        # fp32 sums of d products: d/2 ulp of sum |x r| at most, a few ulp of the row's magnitude in fact
        np.testing.assert_allclose(s, 0.9 * np.abs(y).max(1) / 7, rtol=2e-5)
        v = y / s[:, None]
        q = np.clip(np.rint(v), -7, 7)
        c = codes[b].cpu().numpy().astype(np.float64)
        assert (np.abs(c) <= 7).all()
        off = np.abs(v - (np.floor(v) + 0.5)) > 1e-3  # away from a rounding boundary
        assert (c[off] == q[off]).all()
        e = ((y - c * s[:, None]) ** 2).sum(1)
        np.testing.assert_allclose(err[b, :, 0].cpu().numpy(), e, rtol=1e-4)
        np.testing.assert_allclose(err[b, :, 1].cpu().numpy(), (y * y).sum(1), rtol=1e-4)


def _few_cu_stream(cus):
    """A stream that may use `cus` compute units (None where the runtime has no such streams)."""
    hip = ctypes.CDLL("libamdhip64.so")
    words = (ctypes.c_uint32 * 8)(*([(1 << cus) - 1] + [0] * 7))
    st = ctypes.c_void_p()
    if not hasattr(hip, "hipExtStreamCreateWithCUMask") or hip.hipExtStreamCreateWithCUMask(ctypes.byref(st), 8, words) != 0:
        return None
    return torch.cuda.ExternalStream(st.value)


def test_a_stream_with_fewer_cus_than_a_row_has_tiles():
    n, d = 1000, 4096
    X, R = _problem(1, n, d, seed=9)
    X, R = X.cuda(), R.cuda()
    ws = kt.Workspace("cuda")

    def call():
        dR, rk = torch.full((1, d, d), float("nan"), device="cuda"), torch.full((1, n), float("nan"), device="cuda")
        loss = kt.kt_kurtosis_loss_grad(X, R, dR=dR, row_kurt=rk, workspace=ws)
        return loss.clone(), rk, dR

    ref = call()
    torch.cuda.synchronize()
    st = _few_cu_stream(8)
    if st is None:
        pytest.skip("no streams with a CU mask")
    with torch.cuda.stream(st):
        got = call()
        st.synchronize()
    for a, b in zip(ref, got):
        assert torch.equal(a, b)
