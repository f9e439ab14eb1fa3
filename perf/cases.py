"""Workloads of the positional cross-match, one pass each through the package's public entry points.

A case is a dict of plain values: the entry point, how the sources lie on the sky, the two catalogue sizes, the
radius (arcsec) and the filter precision. Inputs are synthetic (float64 degrees, seeded); the sky models are those of
the repository's own workloads: a small cone, a 10 x 10 degree patch, the full sky with a dense band, polar caps and
the RA seam, and the precision stress (tight clumps, crowded poles and seam, counterparts placed around the radius).
Pairs come back ordered by (a, b), as a program that joins two tables on them wants them, in buffers that the program
keeps; what lies past the pairs found stays zero.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2301_07331_amd as hlc

ARCSEC = 1.0 / 3600.0
D2R = math.pi / 180.0
PRECISION = {"fp32": hlc.HLC_FP32_RECHECK, "fp64": hlc.HLC_FP64}


def listed():
    return [
        # one cone of the batched workload's median size, matched by itself: an interactive query (launches, latency)
        dict(name="cone_2k", entry="xmatch", sky="cone", na=2000, nb=2000, r=1.0, precision="fp32"),
        # a serving loop that may not allocate: the 100,000-source patch, the caller ordering the pairs
        dict(name="noalloc_100k", entry="noalloc", sky="patch", na=100000, nb=100000, r=1.0, precision="fp32"),
        # a patch of a survey against a deeper one, both of odd size, in the FP64 form
        dict(name="patch_ragged_fp64", entry="xmatch", sky="patch", na=299993, nb=1000003, r=1.5, precision="fp64"),
        # per-source error radii (the 3-sigma rule) over a million sources a side
        dict(name="radii_1m", entry="radii", sky="full", na=1000000, nb=1000000, r=2.0, precision="fp32"),
        # one resident partitioned catalogue, new sources partitioned and matched against it
        dict(name="part_2m", entry="part", sky="full", na=2000000, nb=4000000, r=2.0, precision="fp64"),
        # a catalogue against itself (duplicates and neighbours)
        dict(name="self_4m", entry="self", sky="full", na=4000000, nb=4000000, r=5.0, precision="fp32"),
        # the headline workload, both filter precisions
        dict(name="fullsky_10m_fp32", entry="xmatch", sky="full", na=10000000, nb=10000000, r=2.0, precision="fp32"),
        dict(name="fullsky_10m_fp64", entry="xmatch", sky="full", na=10000000, nb=10000000, r=2.0, precision="fp64"),
        # clumps, poles and seam: the sizes of the parity test and of the benchmark
        dict(name="stress_2m_fp64", entry="xmatch", sky="stress", na=2000000, nb=2000000, r=1.0, precision="fp64"),
        dict(name="stress_20m_fp32", entry="xmatch", sky="stress", na=20000000, nb=20000000, r=1.0, precision="fp32"),
        # 10,000 independent cones in one call, another set of cones on every call
        dict(name="batch_10k", entry="batch", sky="jobs", na=10000, nb=2000, r=0.0, precision="fp32"),
        # catalogues in pinned host memory, streamed; the caller keeps each B source's nearest separation
        dict(name="stream_4m_1m", entry="stream", sky="patch", na=4000000, nb=1000000, r=1.0, precision="fp32"),
    ]


def draw(rng):
    def size(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n | 1 if rng.random() < 0.6 else n

    def other(n, lo, hi):
        return min(max(int(round(n * 2.0 ** rng.uniform(-1.5, 1.5))), lo), hi)

    def radius(lo, hi):
        return round(math.exp(rng.uniform(math.log(lo), math.log(hi))), 3)

    precision = rng.choice(["fp32", "fp64"])
    kind = rng.choice(["cone", "patch", "full", "full", "stress", "noalloc", "radii", "part", "self", "batch", "stream"])
    if kind == "cone":
        na = size(500, 50000)
        return dict(entry="xmatch", sky="cone", na=na, nb=other(na, 300, 50000), r=radius(0.5, 5.0), precision=precision)
    if kind == "patch":
        na = size(20000, 3000000)
        return dict(entry="xmatch", sky="patch", na=na, nb=other(na, 10000, 3000000), r=radius(0.5, 5.0),
                    precision=precision)
    if kind == "full":
        na = size(300000, 10000000)
        return dict(entry="xmatch", sky="full", na=na, nb=other(na, 200000, 10000000), r=radius(0.5, 5.0),
                    precision=precision)
    if kind == "stress":
        na = size(1000000, 20000000)
        return dict(entry="xmatch", sky="stress", na=na, nb=na, r=radius(0.5, 1.0), precision=precision)
    if kind == "noalloc":
        na = size(2000, 300000)
        return dict(entry="noalloc", sky="patch", na=na, nb=other(na, 1000, 300000), r=radius(0.5, 2.0),
                    precision=precision)
    if kind in ("radii", "part"):
        na = size(200000, 4000000)
        return dict(entry=kind, sky="full", na=na, nb=other(na, 200000, 4000000), r=radius(1.0, 4.0),
                    precision=precision)
    if kind == "self":
        na = size(200000, 5000000)
        return dict(entry="self", sky="full", na=na, nb=na, r=radius(1.0, 5.0), precision=precision)
    if kind == "batch":
        return dict(entry="batch", sky="jobs", na=size(100, 8000), nb=size(300, 2000), r=0.0, precision=precision)
    na = size(1000000, 8000000)
    return dict(entry="stream", sky="patch", na=na, nb=size(300000, 2000000), r=radius(0.5, 1.5), precision=precision)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Gen:
    """Seeded float64 samples on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 2301073310)

    def u(self, n, lo=0.0, hi=1.0):
        return torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64) * (hi - lo) + lo

    def normal(self, n):
        return torch.randn(n, generator=self.g, device="cuda", dtype=torch.float64)

    def ints(self, n, hi):
        return torch.randint(0, hi, (n,), generator=self.g, device="cuda")

    def perm(self, n):
        return torch.randperm(n, generator=self.g, device="cuda")


def _wrap(ra):
    ra = torch.remainder(ra, 360.0)
    return torch.where(ra >= 360.0, torch.zeros_like(ra), ra)


def _offset(ra, dec, rho, pa):
    """Sources moved by rho degrees along position angle pa (radians)."""
    d, p = dec * D2R, rho * D2R
    sd, cd, sp, cp = torch.sin(d), torch.cos(d), torch.sin(p), torch.cos(p)
    s = (sd * cp + cd * sp * torch.cos(pa)).clamp(-1.0, 1.0)
    dra = torch.atan2(torch.sin(pa) * sp * cd, cp - sd * s)
    return _wrap(ra + dra / D2R), (torch.asin(s) / D2R).clamp(-90.0, 90.0)


def _gauss(g, ra, dec, sigma_as):
    n = ra.numel()
    x, y = g.normal(n) * (sigma_as * ARCSEC), g.normal(n) * (sigma_as * ARCSEC)
    return _offset(ra, dec, torch.hypot(x, y), torch.atan2(x, y))


def _sphere(g, n):
    return g.u(n, 0.0, 360.0), torch.asin(g.u(n, -1.0, 1.0)) / D2R


def _in_patch(g, n):
    return g.u(n, 150.0, 160.0), torch.asin(g.u(n, 0.0, math.sin(10.0 * D2R))) / D2R


def _in_cone(g, ra, dec, radius):
    n = ra.numel()
    rho = torch.acos((1.0 - g.u(n) * (1.0 - torch.cos(radius * D2R))).clamp(-1.0, 1.0)) / D2R
    return _offset(ra, dec, rho, g.u(n, 0.0, 2.0 * math.pi))


def _caps(g, n):
    s = 1.0 - g.u(n) * (1.0 - math.cos(D2R))
    dec = 90.0 - torch.acos(s) / D2R
    return g.u(n, 0.0, 360.0), torch.where(g.u(n) < 0.5, dec, -dec)


def _seam(g, n, half_as):
    return _wrap(g.u(n, -half_as * ARCSEC, half_as * ARCSEC)), torch.asin(g.u(n, -1.0, 1.0)) / D2R


def _band(g, n):
    """The sphere with five times the density within 10 degrees of a great circle (pole at RA 270, Dec +30)."""
    s0 = math.sin(10.0 * D2R)
    inside = g.u(n) < 5.0 * s0 / (5.0 * s0 + 1.0 - s0)
    v = g.u(n, -1.0, 1.0)
    out = torch.where(v >= 0, 1.0, -1.0) * (s0 + v.abs() * (1.0 - s0))
    lat = torch.asin(torch.where(inside, v * s0, out)) / D2R
    # latitude from the plane is 90 degrees less the distance from its pole
    return _offset(torch.full_like(lat, 270.0), torch.full_like(lat, 30.0), 90.0 - lat, g.u(n, 0.0, 2.0 * math.pi))


def _cat(*parts):
    return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])


def _shuffled(g, p):
    k = g.perm(p[0].numel())
    return p[0][k].contiguous(), p[1][k].contiguous()


def _side(g, sky, n, centres):
    if sky == "patch":
        return _in_patch(g, n)
    if sky == "cone":
        return _in_cone(g, torch.full((n,), 75.0, device="cuda", dtype=torch.float64),
                        torch.full((n,), -32.0, device="cuda", dtype=torch.float64),
                        torch.full((n,), 1.0, device="cuda", dtype=torch.float64))
    if sky == "full":
        k = n // 100
        return _cat(_band(g, n - 2 * k), _caps(g, k), _seam(g, k, 1.0))
    n_cl, n_un, n_cap = n // 2, n // 4, n // 8
    k = g.ints(n_cl, centres[0].numel())
    return _cat(_gauss(g, centres[0][k], centres[1][k], 30.0), _sphere(g, n_un), _caps(g, n_cap),
                _seam(g, n - n_cl - n_un - n_cap, 2.0))


# share of B that are counterparts of A sources, and their positional error (arcsec)
COUNTERPARTS = {"cone": (0.3, 0.3), "patch": (0.3, 0.3), "full": (0.4, 0.5), "stress": (0.5, 0.0)}


def _catalogues(case, seed):
    g = _Gen(seed)
    sky, na, nb, r = case["sky"], case["na"], case["nb"], case["r"]
    centres = _sphere(g, max(1, na // 2000)) if sky == "stress" else None
    a = _shuffled(g, _side(g, sky, na, centres))
    if case["entry"] == "self":
        return a, a
    share, sigma = COUNTERPARTS[sky]
    nc = min(int(share * nb), na)
    k = g.perm(na)[:nc]
    if sky == "stress":
        c = _offset(a[0][k], a[1][k], g.u(nc, 0.99 * r * ARCSEC, 1.01 * r * ARCSEC), g.u(nc, 0.0, 2.0 * math.pi))
    else:
        c = _gauss(g, a[0][k], a[1][k], sigma)
    return a, _shuffled(g, _cat(c, _side(g, sky, nb - nc, centres)))


def _job_tables(case, seed):
    """na jobs of median size nb: lognormal sizes, cone radii 0.1 to 2 degrees, r 0.5 to 3 arcsec."""
    q = np.random.Generator(np.random.PCG64(np.random.SeedSequence([2301073310, int(seed)])))
    nj = case["na"]
    na, nb = (np.clip(np.round(np.exp(q.normal(math.log(case["nb"]), 1.0, nj))), 100, 1000000).astype(np.int64)
              for _ in range(2))
    a_off, b_off = np.cumsum(na) - na, np.cumsum(nb) - nb
    r = q.uniform(0.5, 3.0, nj)
    table = hlc.job_table(list(zip(a_off.tolist(), na.tolist(), b_off.tolist(), nb.tolist(), r.tolist())))
    return table, na, nb, r


def _job_sources(na, nb, seed):
    g = _Gen(seed)
    nj = len(na)
    cra, cdec = _sphere(g, nj)
    radius = g.u(nj, 0.1, 2.0)
    ta, tb = torch.from_numpy(na).cuda(), torch.from_numpy(nb).cuda()
    ja = torch.repeat_interleave(torch.arange(nj, device="cuda"), ta)
    jb = torch.repeat_interleave(torch.arange(nj, device="cuda"), tb)
    a = _in_cone(g, cra[ja], cdec[ja], radius[ja])
    b = _in_cone(g, cra[jb], cdec[jb], radius[jb])
    # about 30 % of a job's B sources are counterparts of its A sources (another one each)
    slot = torch.arange(jb.numel(), device="cuda") - (torch.cumsum(tb, 0) - tb)[jb]
    k = torch.nonzero((g.u(jb.numel()) < 0.3) & (slot < ta[jb])).flatten()
    at = (torch.cumsum(ta, 0) - ta)[jb[k]] + slot[k]
    c = _gauss(g, a[0][at], a[1][at], 0.3)
    b[0][k], b[1][k] = c
    return tuple(x.contiguous() for x in a), tuple(x.contiguous() for x in b), ja, jb


def _errors(case, seed):
    """Positional errors (arcsec) of the two catalogues, up to a largest one whose 3-sigma radius is the case's r."""
    g = _Gen(seed + 7919)
    top = case["r"] / (3.0 * math.sqrt(2.0))
    return g.u(case["na"], 0.2 * top, top), g.u(case["nb"], 0.2 * top, top)


def _pairs_expected(case):
    na, nb, r = case["na"], case["nb"], case["r"]
    if case["entry"] == "batch":
        return 0.3 * na * nb * math.exp(0.5) * 0.72
    rr = (r * ARCSEC * D2R) ** 2
    if case["entry"] == "self":
        return 0.5 * na * nb * rr / 4.0 * 3.0
    share, sigma = COUNTERPARTS[case["sky"]]
    nc = min(int(share * nb), na)
    if case["sky"] == "stress":
        return 0.5 * nc + 0.6 * nb * r * r
    if case["entry"] == "radii":
        r *= 0.6
    area = {"cone": math.pi * D2R * D2R, "patch": 100.0 * D2R * D2R, "full": 4.0 * math.pi / 2.4}[case["sky"]]
    return nc * (1.0 - math.exp(-0.5 * (r / sigma) ** 2)) + na * nb * math.pi * rr / area


def work(case):
    """16 B of each source's position in, 16 B of each pair out; a key per source, a great-circle angle per pair."""
    na, nb = case["na"], case["nb"]
    if case["entry"] == "batch":
        na = nb = case["na"] * case["nb"] * math.exp(0.5)
    if case["entry"] == "self":
        nb = 0
    pairs = _pairs_expected(case)
    read = (24 if case["entry"] == "radii" else 16) * (na + nb)
    written = 8 * nb if case["entry"] == "stream" else 16 * pairs
    return {"bytes": float(read + written), "flops": 4.0 * (na + nb) + 50.0 * pairs}


# ---------------------------------------------------------------------------
# a pass
# ---------------------------------------------------------------------------
def _capacity(case):
    """Pairs that the caller's buffers hold."""
    if case["entry"] == "batch":
        return int(case["na"] * case["nb"] * 1.1) + 1024
    return max(1024, (case["na"] + case["nb"]) * (2 if case["sky"] == "stress" else 1) // 2)


def prepare(case, seed):
    s = dict(case)
    s["precision"] = PRECISION[case["precision"]]
    if case["entry"] == "batch":
        s["jobs"], na, nb, _ = _job_tables(case, seed)
        s["a"], s["b"], _, _ = _job_sources(na, nb, seed)
        s["counts"] = torch.zeros(len(na), dtype=torch.int64, device="cuda")
    else:
        s["a"], s["b"] = _catalogues(case, seed)
    if case["entry"] == "radii":
        s["ea"], s["eb"] = _errors(case, seed)
    if case["entry"] == "stream":
        # the catalogues lie in page-locked host memory; the caller keeps a table of nearest separations
        s["a"], s["b"] = (tuple(x.cpu().pin_memory() for x in p) for p in (s["a"], s["b"]))
        s["nearest"] = np.full(case["nb"], np.inf)
        return s
    cap = _capacity(case)
    s["pairs"] = torch.zeros((cap, 2), dtype=torch.int32, device="cuda")
    s["sep"] = torch.zeros(cap, dtype=torch.float64, device="cuda")
    if case["entry"] == "noalloc":
        s["keys"], s["order"] = (torch.zeros(cap, dtype=torch.int64, device="cuda") for _ in range(2))
        s["by_key"] = torch.zeros(cap, dtype=torch.float64, device="cuda")
    if case["entry"] == "part":
        st, s["part"] = hlc.hlc_partition(*s["b"], case["r"])
        _ok(st)
    return s


def _ok(status):
    if status != hlc.HLC_OK:
        raise hlc.HLCError(status)


def run(s):
    entry, prec, r = s["entry"], s["precision"], s["r"]
    if entry == "stream":
        nearest = s["nearest"]

        def sink(pairs, sep, n):
            b = np.ctypeslib.as_array(ctypes.cast(pairs, ctypes.POINTER(ctypes.c_uint32)), shape=(n, 2))[:, 1]
            np.minimum.at(nearest, b, np.ctypeslib.as_array(ctypes.cast(sep, ctypes.POINTER(ctypes.c_double)),
                                                            shape=(n,)))
            return 0

        st, n = hlc.hlc_xmatch_stream(*s["a"], *s["b"], r, sink, precision=prec, ring_pairs=1 << 22)
        _ok(st)
        return nearest, n
    pairs, sep = s["pairs"], s["sep"]
    if entry == "noalloc":
        st, n = hlc.hlc_xmatch_noalloc(*s["a"], *s["b"], r, pairs, sep, precision=prec)
        _ok(st)
        # (this entry point returns a set: the caller orders it)
        order = s["order"][:n]
        torch.sort(pairs[:n].view(torch.int64).flatten(), out=(s["keys"][:n], order))
        torch.index_select(sep[:n], 0, order, out=s["by_key"][:n])
        return s["keys"].view(torch.int32).view(-1, 2), s["by_key"], n
    if entry == "xmatch":
        st, n = hlc.hlc_xmatch(*s["a"], *s["b"], r, pairs, sep, precision=prec, flags=hlc.HLC_SORTED)
    elif entry == "radii":
        st, n = hlc.hlc_xmatch_radii(*s["a"], s["ea"], *s["b"], s["eb"], 3.0, pairs, sep, precision=prec,
                                     flags=hlc.HLC_SORTED)
    elif entry == "self":
        st, n = hlc.hlc_xmatch(*s["a"], *s["a"], r, pairs, sep, precision=prec, flags=hlc.HLC_SELF | hlc.HLC_SORTED)
    elif entry == "part":
        st, part = hlc.hlc_partition(*s["a"], r)
        _ok(st)
        st, n = hlc.hlc_xmatch_part(part, s["part"], r, pairs, sep, precision=prec, flags=hlc.HLC_SORTED)
        part.free()
    else:
        st, n = hlc.hlc_xmatch_batch(s["jobs"], *s["a"], *s["b"], pairs, sep, s["counts"], precision=prec,
                                     flags=hlc.HLC_SORTED)
        _ok(st)
        return pairs, sep, n, s["counts"]
    _ok(st)
    return pairs, sep, n


# ---------------------------------------------------------------------------
# the same results from plain torch in float64
# ---------------------------------------------------------------------------
def _haversine(ra1, dec1, ra2, dec2):
    d = (ra1 - ra2).abs()
    d = torch.where(d > 180.0, 360.0 - d, d)
    s1, s2 = torch.sin(0.5 * D2R * (dec1 - dec2)), torch.sin(0.5 * D2R * d)
    h = s1 * s1 + torch.cos(D2R * dec1) * torch.cos(D2R * dec2) * s2 * s2
    return 2.0 * torch.asin(torch.sqrt(h.clamp(max=1.0))) / D2R * 3600.0


def _join(a, b, rmax, keep):
    """Every (a, b) that `keep(ia, ib, sep)` accepts among the pairs closer than rmax, from a grid of cubic cells."""
    side = max(2.0 * math.sin(0.5 * rmax * ARCSEC * D2R) * (1.0 + 1e-9) + 1e-13, 1e-6)

    def cells(p):
        ra, dec = p[0] * D2R, p[1] * D2R
        xyz = (torch.cos(dec) * torch.cos(ra), torch.cos(dec) * torch.sin(ra), torch.sin(dec))
        return [torch.floor((x + 1.0) / side).to(torch.int64) + 1 for x in xyz]

    def code(x, y, z):
        return (x << 42) | (y << 21) | z

    ca, cb = cells(a), cells(b)
    kb, ob = torch.sort(code(*cb))
    got_a, got_b, got_s = [], [], []
    for at in range(0, a[0].numel(), 1 << 22):
        x, y, z = (c[at:at + (1 << 22)] for c in ca)
        for dx in (-1, 0, 1):
            for dy in (-1, 0, 1):
                lo = torch.searchsorted(kb, code(x + dx, y + dy, z - 1))
                m = torch.searchsorted(kb, code(x + dx, y + dy, z + 1), right=True) - lo
                ia = torch.repeat_interleave(torch.arange(x.numel(), device=x.device), m)
                if not ia.numel():
                    continue
                first = torch.cumsum(m, 0) - m
                ib = ob[lo[ia] + torch.arange(ia.numel(), device=x.device) - first[ia]]
                ia = ia + at
                sep = _haversine(a[0][ia], a[1][ia], b[0][ib], b[1][ib])
                k = torch.nonzero(keep(ia, ib, sep)).flatten()
                got_a.append(ia[k])
                got_b.append(ib[k])
                got_s.append(sep[k])
    if not got_a:
        e = torch.zeros(0, dtype=torch.int64, device=a[0].device)
        return e, e, e.double()
    ia, ib, sep = torch.cat(got_a), torch.cat(got_b), torch.cat(got_s)
    return ia, ib, sep


def _ordered(case, ia, ib, sep):
    n = ia.numel()
    o = torch.argsort((ib << 32) | ia if case["entry"] == "noalloc" else (ia << 32) | ib)
    pairs = torch.zeros((_capacity(case), 2), dtype=torch.int32, device=ia.device)
    seps = torch.zeros(_capacity(case), dtype=torch.float64, device=ia.device)
    pairs[:n] = torch.stack([ia[o], ib[o]], 1).to(torch.int32)
    seps[:n] = sep[o]
    return pairs, seps, n


def exact(case, seed):
    entry, r = case["entry"], case["r"]
    if entry == "batch":
        _, na, nb, rj = _job_tables(case, seed)
        a, b, ja, jb = _job_sources(na, nb, seed)
        rt = torch.from_numpy(rj).cuda()
        ia, ib, sep = _join(a, b, float(rj.max()), lambda i, j, s: (ja[i] == jb[j]) & (s <= rt[ja[i]]))
        return (*_ordered(case, ia, ib, sep), torch.bincount(ja[ia], minlength=len(na)))
    a, b = _catalogues(case, seed)
    if entry == "radii":
        ea, eb = _errors(case, seed)
        ia, ib, sep = _join(a, b, r * (1.0 + 1e-9),
                            lambda i, j, s: s <= 3.0 * torch.sqrt(ea[i] * ea[i] + eb[j] * eb[j]))
    elif entry == "self":
        ia, ib, sep = _join(a, a, r, lambda i, j, s: (s <= r) & (i < j))
    else:
        ia, ib, sep = _join(a, b, r, lambda i, j, s: s <= r)
    if entry == "stream":
        nearest = torch.full((case["nb"],), math.inf, dtype=torch.float64, device="cuda")
        return nearest.scatter_reduce_(0, ib, sep, "amin").cpu().numpy(), int(ia.numel())
    return _ordered(case, ia, ib, sep)
