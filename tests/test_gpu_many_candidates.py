"""Few A sources with many candidates each: the certification's grid before and after the staging grew for them."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb,r", [(40, 30000, 200.0), (2000, 30000, 1500.0), (5000, 20000, 300.0)])
def test_many_candidates(na, nb, r):
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(na)
    sky = [rng.uniform(lo, lo + 1.0, n) for n in (na, nb) for lo in (150.0, 2.0)]
    ref = oracle.xmatch(*sky, r)
    t = [torch.from_numpy(x).cuda() for x in sky]
    pairs = torch.zeros((len(ref) + 8, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(len(ref) + 8, dtype=torch.float64, device="cuda")
    for prec in (0, 1):
        hlc.shutdown()  # (the first call starts from the estimate)
        for _ in range(2):
            st, n = hlc.hlc_xmatch(*t, r, pairs, sep, precision=prec)
            assert (st, n) == (hlc.HLC_OK, len(ref))
            p = pairs[:n].cpu().numpy().astype(np.uint64)
            keys = (p[:, 0] << np.uint64(32)) | p[:, 1]
            o = np.argsort(keys)
            assert np.array_equal(keys[o], ref.keys())
            assert np.abs(sep[:n].cpu().numpy()[o] - ref.sep).max() <= 1e-9
