"""The bucket sort at the sizes where its form changes (one block of 4,096 or 16,384 entries, buckets, the digit sort)
and where a bucket outgrows its block, through every entry point that uses it, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

LAST = 1024 * 1792  # sources of the largest bucket-sorted side


def _sky(kind, n, rng):
    if kind == "even":
        return rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-1, 1, n)))
    if kind == "halo":  # narrow in Dec: many Dec-halo copies
        return rng.uniform(100, 110, n), rng.uniform(20.0, 20.02, n)
    if kind == "line":  # a few Dec values: equal keys in numbers
        return rng.uniform(0, 360, n), rng.integers(-3, 4, n) * 10.0
    ra, dec = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-1, 1, n)))
    m = n // 2  # "crowd": half the sources in one part of the key space
    ra[:m], dec[:m] = rng.uniform(200, 200.3, m), rng.uniform(5, 5.3, m)
    return ra, dec


def _match(entry, hlc, t, r, cap, prec):
    import torch
    pairs = torch.zeros((cap, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(cap, dtype=torch.float64, device="cuda")
    if entry == "part":
        parts = [hlc.hlc_partition(*t[k:k + 2], r) for k in (0, 2)]
        assert all(st == hlc.HLC_OK for st, _ in parts)
        st, n = hlc.hlc_xmatch_part(parts[0][1], parts[1][1], r, pairs, sep, precision=prec)
        for _, p in parts:
            p.free()
    elif entry == "noalloc":
        st, n = hlc.hlc_xmatch_noalloc(*t, r, pairs, sep, precision=prec)
    elif entry == "self":
        st, n = hlc.hlc_xmatch(*t[:2], *t[:2], r, pairs, sep, precision=prec, flags=hlc.HLC_SELF)
    else:
        st, n = hlc.hlc_xmatch(*t, r, pairs, sep, precision=prec)
    assert st == hlc.HLC_OK, hlc.strerror(st)
    p = pairs[:n].cpu().numpy().astype(np.uint64)
    keys = (p[:, 0] << np.uint64(32)) | p[:, 1]
    o = np.argsort(keys)
    return keys[o], sep[:n].cpu().numpy()[o]


@pytest.mark.parametrize("entry", ["xmatch", "part", "noalloc", "self"])
@pytest.mark.parametrize("kind,na,nb,r", [
    ("even", 1, 2048, 2000.0),
    ("even", 2048, 2049, 600.0),
    ("even", 8192, 8193, 300.0),
    ("even", 16383, 16385, 200.0),
    ("halo", 2048, 8192, 20.0),
    ("halo", 8193, 40001, 5.0),
    ("line", 8192, 30000, 60.0),
    ("crowd", 60000, 60001, 2.0),
    ("crowd", 9000, 100000, 2.0),
    ("even", LAST, 100003, 10.0),
    ("even", LAST + 1, LAST, 5.0),
])
def test_bucket_sort(kind, na, nb, r, entry):
    import torch
    import paper_2301_07331_amd as hlc

    if entry == "noalloc" and na + nb > 500000:
        pytest.skip("beyond the fixed scratch")
    if entry == "self" and max(na, nb) > 500000:
        nb, na = nb, min(na, 200000)
    rng = np.random.default_rng(na + nb)
    a, b = _sky(kind, na, rng), _sky(kind, nb, rng)
    k = min(na, nb) // 4
    b[0][:k] = a[0][:k]
    b[1][:k] = np.clip(a[1][:k] + rng.uniform(-r, r, k) / 3600, -90, 90)
    if entry == "self":
        ref = oracle.xmatch(*a, *a, r)
        keep = ref.a < ref.b
        keys, sep = ref.keys()[keep], ref.sep[keep]
    else:
        ref = oracle.xmatch(*a, *b, r)
        keys, sep = ref.keys(), ref.sep
    t = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (*a, *b)]
    for prec in (0, 1):
        got, s = _match(entry, hlc, t, r, len(keys) + 16, prec)
        assert np.array_equal(got, keys)
        assert np.abs(s - sep).max(initial=0.0) <= 1e-9
