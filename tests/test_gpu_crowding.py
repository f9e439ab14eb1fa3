"""Zones thinner than a group's extent and the sub-bin sort of crowded sources: pair sets against the oracle at the
sizes where the sample starts to count crowding, spread evenly and crowded (clumps, a line along the RA seam, a
pole), in whole-sky and smaller frames, with sides of very different size, sorted and shuffled."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

FIRST = 1 << 19  # sources of the larger side from which crowding is counted


def _sky(kind, n, rng):
    ra, dec = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-1, 1, n)))
    if kind == "even":
        return ra, dec
    m = n // 2
    if kind == "clumps":
        c = rng.integers(0, n // 2000 + 1, m)
        dec[:m] = np.clip(dec[c] * 0.9 + rng.normal(0, 30 / 3600, m), -90, 90)
        ra[:m] = (ra[c] + rng.normal(0, 30 / 3600, m)) % 360
    elif kind == "seam":
        ra[:m] = rng.uniform(-2 / 3600, 2 / 3600, m) % 360
    elif kind == "pole":
        dec[:m] = 90 - np.abs(rng.normal(0, 0.2, m))
    elif kind == "patch_clumps":
        ra, dec = rng.uniform(150, 160, n), rng.uniform(0, 10, n)
        c = rng.integers(0, n // 2000 + 1, m)
        ra[:m], dec[:m] = ra[m + c] + rng.normal(0, 30 / 3600, m), dec[m + c] + rng.normal(0, 30 / 3600, m)
        dec = np.clip(dec, -90, 90)
    ra[ra >= 360] = 0.0
    return ra, dec


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind,na,nb,order", [
    ("even", FIRST - 1, FIRST - 1, None),
    ("even", FIRST, FIRST + 1, "dec"),
    ("clumps", FIRST, FIRST, None),
    ("clumps", FIRST - 1, FIRST - 1, None),
    ("clumps", 1000, FIRST + 7, "ra"),
    ("clumps", FIRST + 7, 37, None),
    ("seam", FIRST, FIRST, None),
    ("pole", FIRST, 300001, "dec"),
    ("patch_clumps", FIRST, 400001, None),
])
def test_crowded(kind, na, nb, order, prec):
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(na + nb)
    a, b = _sky(kind, na, rng), _sky(kind, nb, rng)
    k = min(na, nb) // 3  # counterparts
    b[0][:k] = a[0][:k]
    b[1][:k] = np.clip(a[1][:k] + rng.uniform(-2, 2, k) / 3600, -90, 90)
    if order:
        a, b = ([x[np.argsort(s[order == "dec"], kind="stable")] for x in s] for s in (a, b))
    r = 1.5
    ref = oracle.xmatch(*a, *b, r)
    t = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (*a, *b)]
    for _ in range(2):  # the second call starts from what the first one found
        pairs = torch.zeros((len(ref) + 8, 2), dtype=torch.int32, device="cuda")
        sep = torch.zeros(len(ref) + 8, dtype=torch.float64, device="cuda")
        st, n = hlc.hlc_xmatch(*t, r, pairs, sep, precision=prec, flags=hlc.HLC_SORTED)
        assert (st, n) == (hlc.HLC_OK, len(ref))
        p = pairs[:n].cpu().numpy().astype(np.uint64)
        assert np.array_equal((p[:, 0] << np.uint64(32)) | p[:, 1], ref.keys())
        assert np.abs(sep[:n].cpu().numpy() - ref.sep).max(initial=0.0) <= 1e-9
