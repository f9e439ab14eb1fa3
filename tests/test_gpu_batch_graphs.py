"""The batched form's graphs over their lives: autotuned, made again because the pairs outgrew their staging, replayed,
replaced by another job table's and made once more; every call's pairs are the expected ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIDE = 1000  # sources a side of the heavy job, all within r of each other
LIGHT = 19


def _batch(seed, heavy):
    rng = np.random.default_rng(seed)
    n = SIDE if heavy else 8
    a = [np.full(n, 120.0) + rng.uniform(-1e-5, 1e-5, n), np.full(n, 10.0) + rng.uniform(-1e-5, 1e-5, n)]
    b = [x.copy() for x in a]
    jobs, want = [(0, n, 0, n, 3.0)], [np.repeat(np.arange(n), n) * 2 ** 32 + np.tile(np.arange(n), n)]
    for k in range(LIGHT):  # 300 sources a degree apart, each with its counterpart
        ra, dec = 10.0 + k + np.arange(300) % 20 * 1.0, -40.0 + np.arange(300) // 20 * 1.0
        o = len(a[0])
        jobs.append((o, 300, o, 300, 1.0))
        want.append((o + np.arange(300)) * 2 ** 32 + o + np.arange(300))
        for side, d in ((a, 0.0), (b, 1e-4)):
            side[0] = np.concatenate([side[0], ra])
            side[1] = np.concatenate([side[1], dec + d])
    return jobs, a + b, np.concatenate(want)


@pytest.mark.parametrize("prec", ["HLC_FP32_RECHECK", "HLC_FP64"])
def test_graphs(prec):
    import torch
    import paper_2301_07331_amd as hlc

    first, second = _batch(1, True), _batch(2, False)
    cap = len(first[2]) + 100
    pairs = torch.zeros((cap, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(cap, dtype=torch.float64, device="cuda")
    hlc.shutdown()  # (staging sizes of earlier calls)
    for jobs, arrs, want in (first, first, second, first, second):
        t = [torch.from_numpy(x).cuda() for x in arrs]
        cnt = torch.zeros(len(jobs), dtype=torch.int64, device="cuda")
        st, n = hlc.hlc_xmatch_batch(jobs, *t, pairs, sep, cnt, precision=getattr(hlc, prec))
        assert (st, n) == (hlc.HLC_OK, len(want))
        p = pairs[:n].cpu().numpy().astype(np.int64)
        assert np.array_equal(np.sort(p[:, 0] * 2 ** 32 + p[:, 1]), want)
        assert cnt.cpu().tolist() == [len(first[2]) - 300 * LIGHT if jobs is first[0] else 64] + [300] * LIGHT
