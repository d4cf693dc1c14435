"""bf16 rows of m 2^k elements, m > 1, up to 32768, are transformed in one pass: the order-M factor exactly on the matrix
cores, the rest in fp32, ONE rounding to bf16.  So the bound has no intermediate rounding in it: 1e-5 of the row norm for the
fp32 tree plus 2^-8 of the value for the rounding."""
import numpy as np
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


# Paley I and II, Sylvester; one to eight waves at work, M a multiple of 16 or not, 64 and 128 columns, more rows than workgroups
@pytest.mark.parametrize("n,d", [(3, 1536), (70, 2560), (5, 4608), (9, 5120), (40, 5632), (600, 6144), (4, 8192), (3, 9216), (5, 13824),
                                 (530, 14336), (2, 16384), (1, 18432), (3, 20480), (300, 24576), (2, 28672), (2, 27648), (65, 32768)])
@pytest.mark.parametrize("use_signs", [True, False])
def test_one_rounding(n, d, use_signs):
    rows = min(n, 4)  # the oracle's rows: the first ones and the last
    X = ktgen.make_x(n, d, seed=n + d, outlier_cols=3, outlier_scale=40.0, t_frac=0.02, dtype="bf16")
    g = torch.Generator().manual_seed(d)
    store = (torch.randint(0, 2, (d + 1,), generator=g) * 2 - 1).to(torch.int8)
    sd = store.cuda()[1:] if use_signs else None    # any alignment
    Y = kt.kt_hadamard_rows(X.cuda(), signs=sd)
    torch.cuda.synchronize()
    pick = np.unique(np.r_[np.arange(rows), n - 1])
    ref = oracle.hadamard_rows(ktgen.to_f64(X)[pick], store[1:].numpy().astype(np.float64) if use_signs else None)
    got = Y.float().cpu().numpy().astype(np.float64)
    rown = np.linalg.norm(ref, axis=1, keepdims=True)
    assert (np.abs(got[pick] - ref) <= 1e-5 * rown + np.abs(ref) * 2.0 ** -8).all()
    assert np.allclose(np.linalg.norm(got, axis=1), np.linalg.norm(ktgen.to_f64(X), axis=1), rtol=3e-3)


@pytest.mark.parametrize("d", [3072, 14336, 28672])
def test_strided_rows_in_place(d):
    n = 11
    buf = torch.randn(n, d + 72, device="cuda").to(torch.bfloat16)
    X, guard = buf[:, :d], buf[:, d:].clone()
    ref = oracle.hadamard_rows(ktgen.to_f64(X.contiguous()))
    other = torch.empty(n, d + 8, dtype=torch.bfloat16, device="cuda")
    kt.kt_hadamard_rows(X, out=other[:, :d])
    kt.kt_hadamard_rows(X, out=X)
    torch.cuda.synchronize()
    assert torch.equal(other[:, :d], X) and torch.equal(buf[:, d:], guard)
    rown = np.linalg.norm(ref, axis=1, keepdims=True)
    assert (np.abs(ktgen.to_f64(X.contiguous()) - ref) <= 1e-5 * rown + np.abs(ref) * 2.0 ** -8).all()


def test_infinities_and_nan_stay_in_their_row():
    d = 13824  # 108 x 128: the tile has padding rows
    X = torch.ones(5, d, device="cuda", dtype=torch.bfloat16)
    X[1, 77] = float("inf")
    X[3, 4000] = float("nan")
    Y = kt.kt_hadamard_rows(X)
    torch.cuda.synchronize()
    assert torch.isinf(Y[1]).all() and torch.isnan(Y[3]).all()
    assert torch.isfinite(Y[[0, 2, 4]]).all() and torch.equal(Y[0], Y[2]) and torch.equal(Y[0], Y[4])


@pytest.mark.parametrize("n,d", [(2, 1536), (3, 8192), (5, 14336), (3, 28672), (66, 32768)])
@pytest.mark.parametrize("size", [3e37, 1e36, 1e-36, 1e-39])
def test_whole_range_of_bf16(n, d, size):
    """A sum of d values that only fits 32 bits after the division by sqrt(d), and values down to the smallest: bf16 numbers
    below 2^-126 lie 2^-133 apart, so half of that is added to the bound."""
    g = torch.Generator().manual_seed(d)
    X = (torch.randn(n, d, generator=g) * size).to(torch.bfloat16)
    Y = kt.kt_hadamard_rows(X.cuda())
    torch.cuda.synchronize()
    pick = [0, n - 1]
    ref, got = oracle.hadamard_rows(ktgen.to_f64(X)[pick]), Y.cpu().double().numpy()[pick]
    rown = np.linalg.norm(ref, axis=1, keepdims=True)
    assert (np.abs(got - ref) <= 1e-5 * rown + np.abs(ref) * 2.0 ** -8 + 2.0 ** -134).all()


@pytest.mark.parametrize("d", [1536, 14336, 28672])
def test_results_beyond_bf16_are_infinite_and_alone(d):
    """Rows of the largest bf16 value: only column 0 of every segment of 2^k is not zero."""
    top = torch.finfo(torch.bfloat16).max
    Y = kt.kt_hadamard_rows(torch.full((2, d), top, dtype=torch.bfloat16, device="cuda"))
    torch.cuda.synchronize()
    ref, got = oracle.hadamard_rows(np.full((2, d), top)), Y.cpu().double().numpy()
    beyond = np.abs(ref) > 1.01 * top
    assert beyond.any() and np.array_equal(got[beyond], np.sign(ref[beyond]) * np.inf)
    assert (np.abs(got - ref)[~beyond] <= np.abs(ref)[~beyond] * 2.0 ** -8).all()


@pytest.mark.parametrize("n,d", [(5, 1536), (530, 5120), (3, 8192), (4, 14336), (3, 28672), (66, 32768)])
@pytest.mark.parametrize("low,high", [(-1, 1), (-128, 127)])
def test_factors_that_are_not_signs(n, d, low, high):
    """`signs` multiplies, whatever int8 values it holds: 0 drops a channel."""
    g = torch.Generator().manual_seed(d + high)
    X = torch.randn(n, d, generator=g).to(torch.bfloat16)
    f = torch.randint(low, high + 1, (d,), generator=g).to(torch.int8)
    f[0], f[d - 1] = low, 0
    Y = kt.kt_hadamard_rows(X.cuda(), signs=f.cuda())
    ones = torch.ones(d, dtype=torch.int8)
    ones[d - 1] = 3     # one such value anywhere
    Z = kt.kt_hadamard_rows(X.cuda(), signs=ones.cuda())
    torch.cuda.synchronize()
    pick = [0, n - 1]
    for got, factor in ((Y, f), (Z, ones)):
        ref, y = oracle.hadamard_rows(ktgen.to_f64(X)[pick], factor.numpy().astype(np.float64)), got.cpu().double().numpy()[pick]
        rown = np.linalg.norm(ref, axis=1, keepdims=True)
        assert (np.abs(y - ref) <= 1e-5 * rown + np.abs(ref) * 2.0 ** -8).all()


def test_factors_that_are_not_signs_in_place():
    n, d = 600, 6144
    X = torch.randn(n, d, device="cuda").to(torch.bfloat16)
    f = torch.randint(-2, 3, (d,), device="cuda").to(torch.int8)
    Y = kt.kt_hadamard_rows(X, signs=f)
    kt.kt_hadamard_rows(X, signs=f, out=X)
    torch.cuda.synchronize()
    assert torch.equal(X, Y)


# fp32 rows: one kernel or two by size (orders 4, 8, 12, 20, 28 and 108, one row to more than two a workgroup, the last block of 4096 partly
# filled), in place and between wide rows, with signs that are not +-1
@pytest.mark.parametrize("n,d", [(1, 1536), (1, 5120), (600, 5120), (1025, 1536), (3, 8192), (530, 8192), (2, 13824), (63, 14336), (64, 14336), (2, 16384),
                                 (63, 32768), (64, 32768)])
@pytest.mark.parametrize("in_place", [False, True])
def test_fp32_rows(n, d, in_place):
    m, p2, kind = oracle.hadamard_factor(d)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.randn((n, d + 4), generator=g, device="cuda")[:, :d]
    signs = torch.randint(-1, 2, (d,), generator=g, device="cuda").to(torch.int8)
    # the columns of H_d from transforms of unit rows are the oracle's business (test_gpu_hadamard.py); here: few rows against it
    rows = sorted({0, n // 2, n - 1})
    ref = oracle.hadamard_rows(X[rows].cpu().double().numpy(), signs.cpu().double().numpy())
    out = X if in_place else torch.full((n, d + 8), float("nan"), device="cuda")[:, :d]
    kt.kt_hadamard_rows(X, signs=signs, out=out)
    got = out[rows].cpu().double().numpy()
    # d values in a tree of depth log2 p2 and a sum of m: 2^-24 of the row's norm per level
    assert (np.abs(got - ref) <= 1e-5 * np.linalg.norm(ref, axis=1, keepdims=True) + 1e-30).all()
    assert torch.isfinite(out).all()
