"""A workspace too small for the recommended plan costs the host next to nothing: the d = 128 loss fits its number of workgroups to the
bytes it is given, which must not be a search over all of them.  No GPU needed: the calls end at the check of the workspace."""
import time

import pytest

import paper_2503_01483_amd as kt

ADDRESS = 1 << 20  # never read: the workspace is refused first


@pytest.mark.parametrize("batch,n", [(1, 131072), (2, 131072)])
def test_refused_workspace_of_fused_loss(batch, n):
    lib = kt.lib()

    def call(size):
        return lib.kt_kurtosis_loss_grad(ADDRESS, 128, ADDRESS, 128, batch, n, 128, kt.KT_BF16, kt.KT_F32, 0.0, ADDRESS, None, ADDRESS,
                                         ADDRESS, size, None)

    assert call(0) == call(255) == 4  # KT_ERR_WORKSPACE_TOO_SMALL
    t = time.perf_counter()
    for _ in range(20):
        call(255)
    one = (time.perf_counter() - t) / 20
    # one scan over at most 1024 numbers of workgroups is some ten us; one for each of 256 of them was 2 ms
    assert one < 3e-4, one
