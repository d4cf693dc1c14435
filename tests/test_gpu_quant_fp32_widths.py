"""Quantisation figures of fp32 rows that do not fill the registers of their kernel (16 and 32 float4 a lane): the narrowest and wide rows of both.  With
the identity rotation Y = X, so that maxima, thresholds and counts are exact."""
import numpy as np
import pytest
import torch

import ktgen
import oracle
import paper_2503_01483_amd as kt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2176, 3968, 4224, 7168])
@pytest.mark.parametrize("q", [0.98, 1.0])
def test_figures(d, q):
    n = 41
    X = ktgen.make_x(n, d, seed=d, outlier_cols=4, outlier_scale=30.0, t_frac=0.05, dtype="f32").reshape(1, n, d)
    X[0, 3] = 0.0
    out = {k: torch.full((1, n, 2), float("nan"), device="cuda") for k in ("amax", "err_sym", "err_asym")}
    out["threshold"], out["success"] = torch.full((1, n), float("nan"), device="cuda"), torch.full((1,), -1, dtype=torch.int64, device="cuda")
    kt.kt_rotate_quant_metrics(X.cuda(), torch.eye(d, device="cuda").unsqueeze(0), quantile=q, **out)
    o = oracle.quant_metrics(ktgen.to_f64(X[0]), np.eye(d), float(np.float32(q)))
    got = {k: v[0].cpu().numpy() for k, v in out.items()}
    assert np.array_equal(got["amax"], o["amax"]) and np.array_equal(got["threshold"], o["thr"]) and int(got["success"]) == o["success"]
    # squares summed four at a time in fp32, then in fp64
    assert np.allclose(got["err_sym"], o["err_sym"], rtol=2e-6, atol=1e-30)
    assert np.allclose(got["err_asym"], o["err_asym"], rtol=2e-6, atol=1e-30)
