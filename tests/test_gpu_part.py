"""GPU: reusable partitions (hlc_partition / hlc_xmatch_part) against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_same, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hlc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2301_07331_amd as m
    m.load()
    return m


def _run(hlc, A, B, r, prec, cap):
    import torch
    out = torch.empty((cap, 2), dtype=torch.int32, device="cuda")
    sep = torch.empty(cap, dtype=torch.float64, device="cuda")
    st, n = hlc.hlc_xmatch_part(A, B, r, out, sep, precision=prec)
    assert st == hlc.HLC_OK, hlc.strerror(st)
    p = out[:n].cpu().numpy().view(np.uint32).reshape(-1, 2)
    keys = (p[:, 0].astype(np.uint64) << np.uint64(32)) | p[:, 1].astype(np.uint64)
    order = np.argsort(keys)
    return keys[order], sep[:n].cpu().numpy()[order]


@pytest.mark.parametrize("prec", [1, 0])
def test_parts_reuse_both_roles(hlc, prec):
    c = synth.patch_pair(scale=0.5, seed_sub=7)
    # crowd the seam and a pole too
    a2, d2, b2, e2 = synth.adversarial("seam", 3000, 3, 3.0)
    a3, d3, b3, e3 = synth.adversarial("pole", 3000, 4, 3.0)
    a_ra = np.concatenate([c.a_ra, a2, a3]); a_dec = np.concatenate([c.a_dec, d2, d3])
    b_ra = np.concatenate([c.b_ra, b2, b3]); b_dec = np.concatenate([c.b_dec, e2, e3])
    st, PA = hlc.hlc_partition(to_dev(a_ra), to_dev(a_dec), 3.0)
    assert st == hlc.HLC_OK
    st, PB = hlc.hlc_partition(to_dev(b_ra), to_dev(b_dec), 3.0)
    assert st == hlc.HLC_OK
    for r in (3.0, 1.0, 0.25):
        ref = oracle.xmatch(a_ra, a_dec, b_ra, b_dec, r)
        keys, sep = _run(hlc, PA, PB, r, prec, len(ref) + 100)
        assert_same(keys, sep, ref, label=f"A-B r={r}")
        ref = oracle.xmatch(b_ra, b_dec, a_ra, a_dec, r)
        keys, sep = _run(hlc, PB, PA, r, prec, len(ref) + 100)
        assert_same(keys, sep, ref, label=f"B-A r={r}")
    ref = oracle.xmatch(a_ra, a_dec, a_ra, a_dec, 1.0)
    keys, sep = _run(hlc, PA, PA, 1.0, prec, len(ref) + 100)
    assert_same(keys, sep, ref, label="A-A")
    assert np.all(np.isin((np.arange(len(a_ra), dtype=np.uint64) << np.uint64(32)) |
                          np.arange(len(a_ra), dtype=np.uint64), keys))
    PA.free()
    PB.free()


@pytest.mark.parametrize("prec", [1, 0])
def test_part_overflow(hlc, prec):
    """Reused partitions: a capacity below the pair count reports the
    required count and writes true pairs into exactly its slots."""
    import torch
    c = synth.patch_pair(scale=0.3, seed_sub=11)
    ref = oracle.xmatch(c.a_ra, c.a_dec, c.b_ra, c.b_dec, 2.0)
    rk = np.sort(ref.keys())
    st, PA = hlc.hlc_partition(to_dev(c.a_ra), to_dev(c.a_dec), 2.0)
    assert st == hlc.HLC_OK
    st, PB = hlc.hlc_partition(to_dev(c.b_ra), to_dev(c.b_dec), 2.0)
    assert st == hlc.HLC_OK
    cap, pad = len(ref) // 3, 100
    out = torch.full((cap + pad, 2), -7, dtype=torch.int32, device="cuda")
    sep = torch.full((cap + pad,), -7.0, dtype=torch.float64, device="cuda")
    st, n = hlc.hlc_xmatch_part(PA, PB, 2.0, out, sep, precision=prec, capacity=cap)
    assert st == hlc.HLC_E_OVERFLOW and n == len(ref)
    o = out.cpu().numpy()
    assert np.all(o[cap:] == -7) and np.all(sep[cap:].cpu().numpy() == -7.0)
    p = o[:cap].view(np.uint32)
    keys = (p[:, 0].astype(np.uint64) << np.uint64(32)) | p[:, 1].astype(np.uint64)
    assert len(np.unique(keys)) == cap and np.all(np.isin(keys, rk))
    PA.free()
    PB.free()


def test_part_errors(hlc):
    import torch
    g = synth.rng(300, 0)
    ra, dec = synth.uniform_sphere(g, 1000)
    st, P1 = hlc.hlc_partition(to_dev(ra), to_dev(dec), 2.0)
    assert st == hlc.HLC_OK
    st, P2 = hlc.hlc_partition(to_dev(ra), to_dev(dec), 2.0, tuning={"zone_height_arcsec": 500.0})
    assert st == hlc.HLC_OK
    out = torch.empty((10, 2), dtype=torch.int32, device="cuda")
    sep = torch.empty(10, dtype=torch.float64, device="cuda")
    st, _ = hlc.hlc_xmatch_part(P1, P1, 2.5, out, sep)  # radius beyond the halo
    assert st == hlc.HLC_E_INVAL
    st, _ = hlc.hlc_xmatch_part(P1, P2, 1.0, out, sep)  # different geometry
    assert st == hlc.HLC_E_INVAL
    bad = dec.copy()
    bad[10] = 95.0
    st, P3 = hlc.hlc_partition(to_dev(ra), to_dev(bad), 2.0)
    assert st == hlc.HLC_E_INVAL and P3 is None
    e = torch.empty(0, dtype=torch.float64, device="cuda")
    st, P4 = hlc.hlc_partition(e, e, 2.0)
    assert st == hlc.HLC_OK
    st, n = hlc.hlc_xmatch_part(P4, P1, 1.0, out, sep)
    assert st == hlc.HLC_OK and n == 0
    for P in (P1, P2, P4):
        P.free()


@pytest.mark.parametrize("sizes", [(5000, 5000), (5000, 20000), (20000, 5000), (1, 70000)])
def test_part_memory_reuse(hlc, sizes):
    """Partitions built in the memory of freed ones (of the same, a larger or a smaller size, while another part
    lives) match as partitions in fresh memory do."""
    import torch

    rng = np.random.default_rng(11)

    def sky(n):
        return [torch.from_numpy(x).cuda() for x in (rng.uniform(10, 12, n), rng.uniform(-1, 1, n))]

    b = sky(30000)
    st, pb = hlc.hlc_partition(*b, 5.0)
    assert st == hlc.HLC_OK
    stream = torch.cuda.Stream()
    for k, n in enumerate(sizes + sizes):
        a = sky(n)
        torch.cuda.synchronize()
        ref = oracle.xmatch(*[x.cpu().numpy() for x in a + b], 5.0)
        st, pa = hlc.hlc_partition(*a, 5.0, stream=stream if k % 2 else None)
        assert st == hlc.HLC_OK
        pairs = torch.zeros((len(ref) + 8, 2), dtype=torch.int32, device="cuda")
        sep = torch.zeros(len(ref) + 8, dtype=torch.float64, device="cuda")
        st, m = hlc.hlc_xmatch_part(pa, pb, 5.0, pairs, sep, flags=hlc.HLC_SORTED)
        assert (st, m) == (hlc.HLC_OK, len(ref))
        p = pairs[:m].cpu().numpy().astype(np.uint64)
        assert np.array_equal((p[:, 0] << np.uint64(32)) | p[:, 1], ref.keys())
        assert np.abs(sep[:m].cpu().numpy() - ref.sep).max(initial=0.0) <= 1e-9
        pa.free()
    pb.free()


@pytest.mark.parametrize("prec", [1, 0])
@pytest.mark.parametrize("n", [3000, 1835009])  # bucket sort, digit sort
def test_part_ties_after_inputs_change(hlc, n, prec):
    """Pairs exactly at the radius, and an ulp to either side, are decided from the (ra, dec) that a partition keeps, not
    from the caller's arrays, which hold something else by then."""
    rng = np.random.default_rng(n)
    r = 3600.0 * 2.0 ** -10  # arcsec: 2^-10 degrees on a meridian
    a_ra, a_dec = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-0.9, 0.9, n)))
    b_ra, b_dec = rng.uniform(0, 360, n), np.degrees(np.arcsin(rng.uniform(-0.9, 0.9, n)))
    m = 300
    at, bt = rng.choice(n, m, replace=False), rng.choice(n, m, replace=False)
    at[0], bt[1] = n - 1, n - 1
    a_ra[at] = b_ra[bt] = rng.integers(0, 360 * 256, m) * 2.0 ** -8
    a_dec[at] = rng.integers(-50 * 256, 50 * 256, m) * 2.0 ** -8
    far = a_dec[at] + 2.0 ** -10
    b_dec[bt] = np.where(np.arange(m) % 3 == 0, far, np.nextafter(far, np.where(np.arange(m) % 3 == 1, 90.0, -90.0)))
    ref = oracle.xmatch(a_ra, a_dec, b_ra, b_dec, r)
    t = [to_dev(x) for x in (a_ra, a_dec, b_ra, b_dec)]
    (s1, PA), (s2, PB) = hlc.hlc_partition(t[0], t[1], r), hlc.hlc_partition(t[2], t[3], r)
    assert s1 == hlc.HLC_OK and s2 == hlc.HLC_OK
    for x in t:
        x.fill_(1.0)
    keys, sep = _run(hlc, PA, PB, r, prec, len(ref) + 1000)
    assert hlc.last_stats()["n_ties"] > 0
    assert_same(keys, sep, ref, label=f"ties {n}")
    PA.free()
    PB.free()
