"""The largest error radii, from per-block maxima: one large radius at the edges of blocks and strides, signed zeros, and
radii that a call refuses wherever they lie, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


def _call(hlc, a, ea, b, eb):
    import torch
    pairs = torch.zeros((4096, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(4096, dtype=torch.float64, device="cuda")
    st, n = hlc.hlc_xmatch_radii(to_dev(a[0]), to_dev(a[1]), to_dev(ea), to_dev(b[0]), to_dev(b[1]), to_dev(eb), 1.0,
                                 pairs, sep)
    p = pairs[:n].cpu().numpy().view(np.uint32).astype(np.uint64)
    return st, np.sort((p[:, 0] << np.uint64(32)) | p[:, 1])


@pytest.mark.parametrize("n,at", [
    (1, 0),
    (255, 254),
    (2048, 2047),
    (2049, 2048),
    (524288, 0),         # the most blocks, one stride each
    (524288, 524287),
    (524289, 524288),    # a second stride
    (1048577, 1048576),
])
@pytest.mark.parametrize("side", ["a", "b"])
def test_largest_radius(n, at, side):
    import paper_2301_07331_amd as hlc
    rng = np.random.default_rng(n + at)
    big = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-0.9, 0.9, n)))
    # one source of the other side, 20 arcsec north of the one with the large radius
    small = np.array([big[0][at]]), np.array([big[1][at] + 20.0 / 3600.0])
    e_big, e_small = np.full(n, -0.0), np.array([0.0])
    e_big[at] = 25.0
    a, ea, b, eb = (big, e_big, small, e_small) if side == "a" else (small, e_small, big, e_big)
    st, keys = _call(hlc, a, ea, b, eb)
    assert st == hlc.HLC_OK
    want = np.sort(oracle.xmatch_radii(*a, ea, *b, eb, 1.0).keys())
    assert len(want) == 1 and np.array_equal(keys, want)
    for bad in (-1e-300, np.nan, np.inf):
        e_big[at] = bad
        assert _call(hlc, a, ea, b, eb)[0] == hlc.HLC_E_INVAL
