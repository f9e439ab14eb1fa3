"""The batched form's order, job by job in LDS: job sizes at the edges of a block's share, jobs shared by several
blocks, clumps that leave a part of the key range too full, and sizes beyond it (the digit sort), against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SMALL = [1, 2, 255, 895, 896, 897, 1024, 1025, 3000]              # mean below 700: blocks of 1,024
LARGE = [3583, 3584, 3585, 4096, 4097, 9000, 20000, 1, 700]       # blocks of 4,096


def _cone(kind, n, rng):
    ra, dec = 150.0 + rng.uniform(-0.1, 0.1, n), 20.0 + rng.uniform(-0.1, 0.1, n)
    if kind == "clump":  # most sources in a few keys
        m = n - n // 8
        ra[:m], dec[:m] = 150.03 + rng.uniform(-1e-7, 1e-7, m), 20.01 + rng.uniform(-1e-5, 1e-5, m)
    elif kind == "point":  # most sources of one key
        m = n - n // 8
        ra[:m], dec[:m] = 150.03, 20.01
    elif kind == "flat":  # one zone row, many Dec-halo copies
        dec = 20.0 + rng.uniform(-2e-4, 2e-4, n)
    return ra, dec


def _run(hlc, sizes_a, sizes_b, kind, r, prec, rng):
    import torch
    sizes_a, sizes_b = [*sizes_a, *[5] * 16], [*sizes_b, *[6] * 16]  # (fewer than 16 jobs: the digit sort)
    a = [_cone("even" if kind in ("clump", "point") else kind, n, rng) for n in sizes_a]
    b = [_cone(kind, n, rng) for n in sizes_b]
    jobs, oa, ob, want, counts = [], 0, 0, [], []
    for (ra, da), (rb, db) in zip(a, b):
        jobs.append((oa, len(ra), ob, len(rb), r))
        n = 0
        if len(ra) and len(rb):
            res = oracle.xmatch(ra, da, rb, db, r)
            n = len(res)
            want.append(((res.a.astype(np.uint64) + np.uint64(oa)) << np.uint64(32))
                        | (res.b.astype(np.uint64) + np.uint64(ob)))
        counts.append(n)
        oa, ob = oa + len(ra), ob + len(rb)
    want = np.sort(np.concatenate(want))
    arrs = [torch.from_numpy(np.concatenate([c[k] for c in side])).cuda() for side in (a, b) for k in (0, 1)]
    cap = len(want) + 1000
    pairs = torch.zeros((cap, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(cap, dtype=torch.float64, device="cuda")
    cnt = torch.zeros(len(jobs), dtype=torch.int64, device="cuda")
    for _ in range(3):  # the second and third replay the captured graph
        st, n = hlc.hlc_xmatch_batch(jobs, *arrs, pairs, sep, cnt, precision=prec,
                                     tuning={"zone_height_factor": 1.0, "batch_tile": 1024, "batch_blocks_per_cu": 4})
        assert st == hlc.HLC_OK, hlc.strerror(st)
        p = pairs[:n].cpu().numpy().view(np.uint32).astype(np.uint64)
        assert np.array_equal(np.sort((p[:, 0] << np.uint64(32)) | p[:, 1]), want)
        assert np.array_equal(cnt.cpu().numpy(), counts)


@pytest.mark.parametrize("prec", ["HLC_FP32_RECHECK", "HLC_FP64"])
@pytest.mark.parametrize("kind,sizes_a,sizes_b,r", [
    ("even", SMALL, SMALL[::-1], 10.0),
    ("even", LARGE, LARGE[::-1], 5.0),
    ("flat", SMALL, SMALL[::-1], 1.0),
    ("flat", LARGE, LARGE[::-1], 1.0),
    ("clump", [400] * 9, [1024, 1025, 5000, 0, 7, 900, 1, 2, 3], 5.0),
    ("clump", [300] * 4, [4096, 4097, 40000, 9000], 5.0),
    ("point", [20] * 4, [4096, 4097, 40000, 9000], 5.0),
    ("even", [3, 500], [57360, 100], 5.0),        # a job read 20 times
    ("even", [3, 500], [57361, 100], 5.0),        # 21 times: the digit sort
    ("even", [3] * 301, [262144] + [3584] * 300, 2.0),  # the largest job ordered in LDS
    ("even", [3] * 301, [262145] + [3584] * 300, 2.0),
])
def test_job_order(kind, sizes_a, sizes_b, r, prec):
    import paper_2301_07331_amd as hlc
    rng = np.random.default_rng(len(kind) * 1000 + sum(sizes_b) % 997)
    _run(hlc, sizes_a, sizes_b, kind, r, getattr(hlc, prec), rng)
