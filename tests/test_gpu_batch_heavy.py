"""Batches in which some jobs' sources have many counterparts each, scattered among ordinary jobs: their groups are
taken first, every pair once."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["HLC_FP32_RECHECK", "HLC_FP64"])
@pytest.mark.parametrize("njobs,heavy,size,extent,dec", [
    (60, 9, 900, 10.0, 20.0),     # about 28 pairs a source: listed
    (60, 60, 300, 6.0, -50.0),    # every group
    (60, 1, 17, 1.0, 5.0),        # two groups of one job
    (40, 7, 700, 22.0, 60.0),     # about 4.5 a source: some groups either way
    (40, 5, 500, 8.0, 89.99),     # whole-circle frames
])
def test_heavy_jobs(njobs, heavy, size, extent, dec, prec):
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(njobs * heavy + size)
    pick = set(rng.choice(njobs, heavy, replace=False).tolist())
    jobs, a, b, want, counts = [], [], [], [], []
    oa = ob = 0
    for j in range(njobs):
        sides = []
        for n in ((size, size + 3) if j in pick else (200, 190)):
            half = (extent if j in pick else 3600.0) / 7200
            de = np.clip(dec + rng.uniform(-half, half, n), -90, 90)
            ra = np.mod(5.0 * j + rng.uniform(-half, half, n) / max(np.cos(np.radians(dec)), 1e-3), 360.0)
            sides.append((ra, de))
        ref = oracle.xmatch(*sides[0], *sides[1], 1.0)
        want.append(((ref.a.astype(np.uint64) + np.uint64(oa)) << np.uint64(32)) | (ref.b.astype(np.uint64) + np.uint64(ob)))
        counts.append(len(ref))
        jobs.append((oa, len(sides[0][0]), ob, len(sides[1][0]), 1.0))
        a.append(sides[0])
        b.append(sides[1])
        oa, ob = oa + len(sides[0][0]), ob + len(sides[1][0])
    want = np.sort(np.concatenate(want))
    t = [torch.from_numpy(np.concatenate([s[k] for s in side])).cuda() for side in (a, b) for k in (0, 1)]
    pairs = torch.zeros((len(want) + 100, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(len(want) + 100, dtype=torch.float64, device="cuda")
    cnt = torch.zeros(njobs, dtype=torch.int64, device="cuda")
    for _ in range(3):
        st, n = hlc.hlc_xmatch_batch(jobs, *t, pairs, sep, cnt, precision=getattr(hlc, prec),
                                     tuning={"zone_height_factor": 1.0, "batch_tile": 1024, "batch_blocks_per_cu": 4})
        assert (st, n) == (hlc.HLC_OK, len(want))
        p = pairs[:n].cpu().numpy().view(np.uint32).astype(np.uint64)
        assert np.array_equal(np.sort((p[:, 0] << np.uint64(32)) | p[:, 1]), want)
        assert cnt.cpu().tolist() == counts
