"""Crowded calls among others, small ones that do not look at the crowding and large ones that are not crowded: what one
call leaves to the next changes no pair."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sky(kind, n, rng):
    ra, dec = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-1, 1, n)))
    if kind == "crowded":  # half the sources in 200 clumps of about an arcminute
        m, c = n // 2, rng.integers(0, 200, n // 2)
        ra[:m] = np.mod(1.8 * c + rng.normal(0, 0.01, m), 360.0)
        dec[:m] = -60.0 + 0.6 * c + rng.normal(0, 0.01, m)
    k = rng.permutation(n)
    return ra[k], dec[k]


def test_crowd_changes():
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(4)
    skies = {}
    for name, kind, n in (("crowded", "crowded", 2000003), ("even", "even", 2000001), ("small", "even", 5001),
                          ("middle", "crowded", 700001)):
        skies[name] = [torch.from_numpy(x).cuda() for s in (0, 1) for x in _sky(kind, n, rng)]

    def run(name, prec):
        pairs = torch.zeros((6000000, 2), dtype=torch.int32, device="cuda")
        st, n = hlc.hlc_xmatch(*skies[name], 2.0, pairs, None, precision=prec, flags=hlc.HLC_NO_SEP)
        assert st == hlc.HLC_OK, hlc.strerror(st)
        p = pairs[:n].to(torch.int64)
        return torch.sort(p[:, 0] * 2 ** 32 + p[:, 1]).values

    for prec in (0, 1):
        want = {}
        for name in skies:
            hlc.shutdown()
            want[name] = run(name, prec)
            assert len(want[name]) > 0 or name == "small"
        for name in ("crowded", "small", "crowded", "even", "crowded", "middle", "crowded", "crowded", "small", "even",
                     "even", "crowded"):
            assert torch.equal(run(name, prec), want[name]), name
