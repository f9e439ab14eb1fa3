"""HLC_SORTED where the buckets are largest: blocks of 12,288 pairs, and a source of more pairs than a bucket may hold
(digit sort), below and above the number of pairs that is ordered before the host knows it."""
import numpy as np
import pytest

from tests.test_gpu_pair_order import SEP_TOL, _expected, _sky

pytestmark = pytest.mark.gpu

CASES = {
    "largest_blocks": [(6, 2, 8000)],                                # 12 buckets of 8,000
    "largest_blocks_and_rounds": [(6, 2, 8000), (1, 1, 20000)],
    "bucket_too_large": [(20000, 1, 1), (1, 1, 66000)],
    "bucket_too_large_many": [(70000, 1, 15), (1, 1, 69000)],        # more than a million pairs
    "bucket_just_fits": [(20000, 1, 1), (1, 1, 60000)],
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_pair_order_limits(case):
    import torch
    import paper_2301_07331_amd as hlc

    a, b = _sky(CASES[case], np.random.default_rng(7))
    ia, ib, sep = _expected(a, b)
    n = len(ia)
    t = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (a[0], a[1], b[0], b[1])]
    for with_sep in (True, False):
        pairs = torch.full((n + 3, 2), -7, dtype=torch.int32, device="cuda")
        out = torch.full((n + 3,), -7.0, dtype=torch.float64, device="cuda")
        flags = hlc.HLC_SORTED | (0 if with_sep else hlc.HLC_NO_SEP)
        st, got = hlc.hlc_xmatch(*t, 1.0, pairs, out if with_sep else None, flags=flags)
        assert (st, got) == (hlc.HLC_OK, n)
        p = pairs.cpu().numpy()
        assert np.array_equal(p[:n, 0], ia) and np.array_equal(p[:n, 1], ib)
        assert (p[n:] == -7).all()
        o = out.cpu().numpy()
        assert (o[n:] == -7.0).all()
        if with_sep:
            assert np.abs(o[:n] - sep).max() <= SEP_TOL
