"""Calls whose footprint changes from one to the next, on both sides of the size above which a sample goes first: the
whole sphere, a patch, and a patch whose sample misses its farthest sources."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sky(kind, n, rng):
    if kind == "full":
        return [rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-1, 1, n)))]
    ra, dec = rng.uniform(150, 160, n), rng.uniform(0, 10, n)
    if kind == "outlier":  # one source far off the rest
        ra[n // 2 + 77], dec[n // 2 + 77] = 171.0, -33.0
    return [ra, dec]


@pytest.mark.parametrize("n", [1 << 20, (1 << 21) + 1])
def test_frame_changes(n):
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(n)
    skies = {}
    for kind in ("full", "patch", "outlier"):
        a = _sky(kind, n, rng)
        k = rng.permutation(n)
        b = [a[0][k], np.clip(a[1][k] + 2e-5, -90, 90)]  # a counterpart 0.072 arcsec away for each
        skies[kind] = ([torch.from_numpy(x).cuda() for x in (*a, *b)], torch.from_numpy(k).cuda())
    pairs = torch.zeros((2 * n, 2), dtype=torch.int32, device="cuda")
    hlc.shutdown()
    for kind in ("full", "patch", "full", "patch", "patch", "outlier", "patch", "full", "outlier", "full", "full"):
        t, k = skies[kind]
        st, m = hlc.hlc_xmatch(*t, 0.1, pairs, None, flags=hlc.HLC_NO_SEP)
        assert st == hlc.HLC_OK, hlc.strerror(st)
        p = pairs[:m].to(torch.int64)
        own = p[k[p[:, 1]] == p[:, 0]]  # each source with its counterpart, once
        assert len(own) == n and len(torch.unique(own[:, 0])) == n
        # the others: neighbours within the radius, a few of this density
        assert m - n < n // 1000
