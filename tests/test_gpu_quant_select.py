"""The quantile threshold where the bin of its order statistic (2048 equal steps up to the row's largest magnitude) and the next
occupied one hold 1, 63, 64, 65 and more values: up to 64 they are ranked against each other, beyond the radix select takes the row.  Also
rows whose squares overflow, of tiny values, of zeros, and with the statistic in the first and the last bin.  With the identity
rotation and fp32 activations Y = X, so the threshold is bit-exact."""
import numpy as np
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


def _rows(d, q, g):
    k = int(np.floor(float(np.float32(q)) * (d - 1)))
    base = torch.sort(torch.rand(d, generator=g) * 0.2 + 0.01).values
    rows = []
    for close, other in ((1, 1), (2, 0), (62, 1), (63, 1), (64, 0), (64, 1), (32, 32), (33, 32), (100, 5)):
        # `close` values about rank k within a bin, `other` ones in the next occupied bin, above them spread ones
        r = base.clone()
        lo = max(0, k - close // 2)
        r[lo:lo + close] = 0.5 + 1e-6 * torch.rand(min(close, d - lo), generator=g)
        r[lo + close:lo + close + other] = 0.6 + 1e-6 * torch.rand(max(0, min(other, d - lo - close)), generator=g)
        rest = d - lo - close - other
        if rest > 0:
            r[lo + close + other:] = 0.7 + 0.3 * torch.arange(1, rest + 1) / rest
        rows.append(r)
    rows += [base * 1e25, base * 1e-33, torch.zeros(d), torch.full((d,), 1e-4).index_fill(0, torch.tensor([3]), 1.0),
             torch.ones(d).index_fill(0, torch.tensor([0, 1]), 1e-6)]
    return torch.stack(rows)


@pytest.mark.parametrize("d", [256, 1152, 4096])
@pytest.mark.parametrize("q", [0.98, 0.5, 0.9999])
def test_threshold(d, q):
    g = torch.Generator().manual_seed(d)
    X = _rows(d, q, g)
    X = X[:, torch.randperm(d, generator=g)] * torch.where(torch.rand(X.shape, generator=g) < 0.5, -1.0, 1.0)
    q = float(np.float32(q))
    thr = torch.full((1, len(X)), float("nan"), device="cuda")
    kt.kt_rotate_quant_metrics(X.unsqueeze(0).cuda(), torch.eye(d, device="cuda").unsqueeze(0), quantile=q, threshold=thr)
    torch.cuda.synchronize()
    want = oracle.quant_metrics(ktgen.to_f64(X), np.eye(d), q)["thr"]
    assert np.array_equal(thr[0].cpu().numpy(), want)


def test_success_counts():
    """Few and many rows a workgroup, several problems."""
    for batch, n, d in ((1, 1, 256), (3, 7, 384), (2, 20011, 256)):
        g = torch.Generator(device="cuda").manual_seed(n)
        X = torch.randn((batch, n, d), generator=g, device="cuda").bfloat16()
        X[:, ::3, 5] = 40.0
        R = torch.stack([ktgen.random_orthogonal(d, seed=b) for b in range(batch)]).cuda()
        amax = torch.empty((batch, n, 2), device="cuda")
        count = torch.full((batch,), -1, dtype=torch.int64, device="cuda")
        kt.kt_rotate_quant_metrics(X, R, amax=amax, success=count)
        assert torch.equal(count, (amax[..., 1] < amax[..., 0]).sum(1))
