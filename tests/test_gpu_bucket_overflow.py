"""A bucket that outgrows its block, with the other side of the call in one block, in buckets, or crowded as well: the
call falls back to the digit sort and its pairs are the oracle's, through every entry point and on one or two streams."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _sky(n, crowded, rng):
    ra, dec = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-1, 1, n)))
    if crowded:  # half the sources in one 8,192th of the key space
        m = n // 2
        ra[:m], dec[:m] = 200.0 + rng.uniform(-1e-3, 1e-3, m), 5.0 + rng.uniform(-1e-3, 1e-3, m)
    return ra, dec


@pytest.mark.parametrize("entry", ["xmatch", "profile", "part", "noalloc"])
@pytest.mark.parametrize("na,nb,crowded", [
    (2000, 100000, (False, True)),    # one block and buckets: two streams
    (100000, 2000, (True, False)),
    (60000, 100000, (True, True)),    # both in buckets: one stream
    (100000, 60000, (False, True)),
])
def test_bucket_overflow(na, nb, crowded, entry):
    import torch
    import paper_2301_07331_amd as hlc

    r = 0.05
    rng = np.random.default_rng(na)
    a, b = _sky(na, crowded[0], rng), _sky(nb, crowded[1], rng)
    k = min(na, nb) // 4
    b[0][-k:] = a[0][-k:]
    b[1][-k:] = np.clip(a[1][-k:] + rng.uniform(-r, r, k) / 3600, -90, 90)
    ref = oracle.xmatch(*a, *b, r)
    t = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (*a, *b)]
    cap = len(ref) + 16
    pairs = torch.zeros((cap, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(cap, dtype=torch.float64, device="cuda")
    for prec in (0, 1):
        hlc.shutdown()  # (nothing known of earlier calls: the first try takes the buckets)
        if entry == "part":
            parts = [hlc.hlc_partition(*t[i:i + 2], r) for i in (0, 2)]
            assert all(st == hlc.HLC_OK for st, _ in parts)
            st, n = hlc.hlc_xmatch_part(parts[0][1], parts[1][1], r, pairs, sep, precision=prec)
            for _, p in parts:
                p.free()
        elif entry == "noalloc":
            st, n = hlc.hlc_xmatch_noalloc(*t, r, pairs, sep, precision=prec)
        else:
            flags = hlc.HLC_PROFILE if entry == "profile" else 0
            st, n = hlc.hlc_xmatch(*t, r, pairs, sep, precision=prec, flags=flags)
        assert st == hlc.HLC_OK, hlc.strerror(st)
        p = pairs[:n].cpu().numpy().astype(np.uint64)
        keys = (p[:, 0] << np.uint64(32)) | p[:, 1]
        o = np.argsort(keys)
        assert np.array_equal(keys[o], ref.keys())
        assert np.abs(sep[:n].cpu().numpy()[o] - ref.sep).max(initial=0.0) <= 1e-9
