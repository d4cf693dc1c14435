"""The ranges of tokens that fp32 dR is summed over: as many as 128 x 128 tiles need to fill the chip (four to a CU), each of at least
eight slabs of 32 tokens, and no longer than that asks for unless four waves share a range.  The workspace holds a d x d partial of each, so its
size tells their number.  No GPU needed."""
import pytest

import paper_2503_01483_amd as kt

CUS = 256


def _ranges(batch, n, d):
    tokens = -(-n // 128) * 128
    bytes_ = kt.kt_workspace_bytes(kt.KT_OP_LOSS_GRAD, batch, n, d, kt.KT_F32)
    # R^T, then Y (dL/dY over it), then the partials; the loss sums are less than one partial
    return (bytes_ - 4 * batch * tokens * d) // (4 * batch * d * d) - 1


@pytest.mark.parametrize("batch,d", [(1, 128), (2, 256), (1, 384), (1, 512), (2, 512), (1, 640), (2, 768), (1, 1024), (2, 1024), (1, 2048)])
def test_no_range_is_longer_than_asked_for(batch, d):
    for n in (300, 1000, 2048, 2400, 3000, 4096, 5000, 7777, 10007, 16384):
        slabs = -(-n // 128) * 4
        tiles = (d // 128) ** 2 * batch
        want = max(1, min(-(-4 * CUS // tiles), slabs // 8))
        length = -(-slabs // want)
        asked = -(-slabs // length)
        got = max(1, _ranges(batch, n, d))
        if (d // 32) ** 2 * batch * asked <= 2 * CUS:  # four waves share a range
            length = -(-length // 4) * 4
            asked = -(-slabs // length)
        assert got == asked, (batch, n, d)
