"""The coarse key index at entry counts where the wave-wide search splits exactly (multiples of 65) and beside them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [0, 8, 30])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 66, 129, 130, 131, 4224, 4225, 4226, 65 * 64 * 3, 65 * 65 * 2])
def test_every_source_meets_itself(n, bins):
    """n sources 1/64 degree of RA apart along the equator, against themselves: n pairs, none lost at an end."""
    import torch
    import paper_2301_07331_amd as hlc

    ra = torch.arange(n, dtype=torch.float64, device="cuda") / 64.0 + 0.25
    dec = torch.zeros(n, dtype=torch.float64, device="cuda")
    pairs = torch.zeros((n + 4, 2), dtype=torch.int32, device="cuda")
    sep = torch.ones(n + 4, dtype=torch.float64, device="cuda")
    for prec in (0, 1):
        st, m = hlc.hlc_xmatch(ra, dec, ra, dec, 1.0, pairs, sep, precision=prec, flags=hlc.HLC_SORTED,
                               tuning=dict(ra_bins_log2=bins))
        assert (st, m) == (hlc.HLC_OK, n)
        want = torch.arange(n, dtype=torch.int32, device="cuda")
        assert (pairs[:n, 0] == want).all() and (pairs[:n, 1] == want).all() and (sep[:n] == 0.0).all()
