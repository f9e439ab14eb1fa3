"""hlc_xmatch_noalloc takes calls up to the sizes that its scratch has always held: the largest of several shapes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb,ra,dec,prec", [
    (873728, 873728, (0.0, 360.0), (-90.0, 90.0), "HLC_FP32_RECHECK"),
    (2041728, 204172, (0.0, 360.0), (-90.0, 90.0), "HLC_FP32_RECHECK"),
    (721472, 721472, (0.0, 360.0), (-90.0, 90.0), "HLC_FP64"),
    (98944, 989440, (0.0, 360.0), (-90.0, 90.0), "HLC_FP64"),
    (98944, 989440, (100.0, 100.02), (-85.0, 85.0), "HLC_FP64"),  # a meridian: the most zones
])
def test_largest_calls(na, nb, ra, dec, prec):
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(na)
    t = [torch.from_numpy(rng.uniform(*lim, n)).cuda() for n in (na, nb) for lim in (ra, dec)]
    out = []
    for call in (hlc.hlc_xmatch, hlc.hlc_xmatch_noalloc):
        pairs = torch.zeros((200000, 2), dtype=torch.int32, device="cuda")
        sep = torch.zeros(200000, dtype=torch.float64, device="cuda")
        st, n = call(*t, 0.5, pairs, sep, precision=getattr(hlc, prec))
        assert st == hlc.HLC_OK, hlc.strerror(st)
        out.append(torch.sort(pairs[:n, 0].to(torch.int64) * 2 ** 32 + pairs[:n, 1]).values)
    assert torch.equal(*out)


def test_largest_call_after_many_candidates():
    """What an earlier call wanted room for does not refuse a call that fits."""
    import torch
    import paper_2301_07331_amd as hlc

    rng = np.random.default_rng(8)
    a = [torch.from_numpy(rng.uniform(20.0, 20.001, 128)).cuda() for _ in range(4)]
    b = [torch.from_numpy(rng.uniform(*lim, 721472)).cuda() for lim in ((0.0, 360.0), (-90.0, 90.0)) * 2]
    pairs = torch.zeros((200000, 2), dtype=torch.int32, device="cuda")
    sep = torch.zeros(200000, dtype=torch.float64, device="cuda")
    for t, r in ((a, 2.0), (b, 0.5)):
        st, n = hlc.hlc_xmatch_noalloc(*t, r, pairs, sep, precision=hlc.HLC_FP64)
        assert st == hlc.HLC_OK, hlc.strerror(st)
