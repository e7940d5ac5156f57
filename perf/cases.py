"""The work that a user of this library has it do, as measurable cases.

Every case is a whole user-visible unit: pairs already in hand go in, the window's report (or
reports) comes out, through the package's public classes and with the library's default launch
settings.  Reports are whole numbers (ip, z0, est, flags), sorted by ip, so they are compared
exactly.  Inputs are made on the GPU from the seed alone: sources whose peer counts follow a
truncated Zipf law, peers drawn with repetition from each source's peers (about 30 % duplicates in
a full window), and planted hosts with distinct peers, in random order, as in `synth_traffic`'s
workloads, whose sketch sizes and traffic shapes these are.
"""
import math
import random

import numpy as np
import torch

import paper_1901_07306_amd as spd

DEV = "cuda"
THETA, SR, A, LOG2K = 1024, 4, 2, 12          # the values of every configuration of this repository
# (r, log2lc): SEAV and LDCA from 128 KiB + 4 MiB (plain_1m) to 16 MiB + 128 MiB (routers_8x16m)
SKETCHES = [(6, 12), (8, 13), (10, 14), (12, 15), (14, 16), (15, 17)]


def _case(name, kind, n, sketch, sources, planted, plo, phi, **kw):
    c = dict(kind=kind, n=n, r=sketch[0], log2lc=sketch[1], lr=2, sources=sources, planted=planted, plo=plo, phi=phi)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a quiet router's window, or one serving batch of the smallest size: latency and launches
        _case("window_4k", "window", 4096, (6, 12), 500, 1, 1200, 1200),
        # a short window of an edge router: still below the default direct/binned crossover
        _case("window_200k", "window", 200_003, (6, 12), 12_000, 6, 2000, 2000),
        # the 1,000,000-pair window of the plain_1m workload
        _case("window_1m", "window", 1_000_000, (6, 12), 50_000, 20, 2000, 2000),
        # an ordinary core-router window with the large sketch, ragged length
        _case("window_5m", "window", 5_000_011, (14, 16), 300_000, 60, 1024, 20000),
        # the 64 Mi-pair window of the plain_64m workload (the benchmark's headline)
        _case("window_64m", "window", 64 << 20, (14, 16), 2_000_000, 500, 1024, 20000),
        # a scan attack: a few hosts send a large share of the window's pairs, the traffic that
        # super-point detection is for
        _case("attack_8m", "window", 8 << 20, (14, 16), 400_000, 4, 1 << 20, 1 << 20),
        # one stream keyed by source and by destination in one call, a report of each
        _case("both_3m", "both", 3_000_000, (12, 15), 150_000, 30, 1024, 20000),
        # the distributed form: 8 routers of 16 Mi pairs scanned in one call and merged, a global
        # report, the routers' sketches started anew
        _case("routers_8x16m", "routers", 16 << 20, (15, 17), 4_000_000, 300, 1024, 20000, routers=8),
        # a slice of the sliding_300x1m workload in steady state: slide, scan, report of the last 60
        # slices, with 8-bit AT counters
        _case("sliding_1m", "sliding", 1_000_000, (14, 16), 1_000_000, 200, 35, 70, slices=60, counter=0),
        # the same with exact 16-bit stamps, a smaller sketch and smaller slices
        _case("sliding_100k_stamps", "sliding", 100_003, (10, 14), 100_000, 40, 35, 70, slices=60, counter=1),
        # pairs in page-locked host memory (the watch point's buffered copy to the GPU)
        _case("host_8m", "host", 8_000_001, (14, 16), 400_000, 60, 1024, 20000),
        # the serving loop: 16 routers' uneven batches as fast as they can be submitted, one window each
        _case("serving_16x4m", "serving", 4 << 20, (14, 16), 200_000, 60, 1024, 20000, routers=16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["window", "window", "window", "noalloc", "both", "routers", "sliding", "host", "serving"])
    sketch = rng.choice(SKETCHES)
    cap = 1 << (sketch[1] + 10)   # a column of the LDCA takes about k / 4 distinct pairs
    kw = {}
    if kind == "window":
        n = _log_uniform(rng, 4096, min(cap, 64 << 20))
    elif kind == "both":
        n = _log_uniform(rng, 4096, min(cap, 16 << 20))
    elif kind == "host":
        n = _log_uniform(rng, 4096, min(cap, 8 << 20))
    elif kind == "noalloc":       # the allocation-free scan
        n = _log_uniform(rng, 4096, min(cap, 16 << 20))
    elif kind == "routers":
        kw["routers"] = rng.randint(2, 8)
        n = _log_uniform(rng, 4096, min(cap, 64 << 20) // kw["routers"])
    elif kind == "sliding":
        kw["slices"] = rng.choice([10, 60, 60, 120])
        kw["counter"] = rng.randint(0, 1)
        n = _log_uniform(rng, 4096, min(cap // 60, 1_000_000))
    else:
        sketch = rng.choice(SKETCHES[2:5])
        kw["routers"] = rng.randint(2, 16)
        n = _log_uniform(rng, 1 << 16, min(1 << (sketch[1] + 10), 4 << 20))
    if kind == "sliding":
        planted, plo, phi = max(1, min(200, n // 5000)), max(35, 1200 // kw["slices"]), max(70, 2400 // kw["slices"])
    else:
        planted, plo, phi = max(1, min(500, n // 20_000)), 1100, (20000 if n > 1 << 21 else 2000)
        if kind == "window" and rng.random() < 0.2 and n > 100_000:   # a scan attack
            planted, plo, phi = 4, n // 8, n // 8
    c = _case(None, kind, n, sketch, max(100, n // 30), planted, plo, phi, **kw)
    c["lr"] = rng.choice([2, 2, 3])
    return c


# ------------------------------------------------------------------------------ inputs
def _gen(seed, *stream):
    g = torch.Generator(device=DEV)
    key = 0x9E3779B97F4A7C15
    for s in (seed,) + stream:
        key = (key ^ (int(s) + 0x7F4A7C15)) * 0xBF58476D1CE4E5B9 % (1 << 63)
        key ^= key >> 31
    g.manual_seed(key)
    return g


def _ips(g, n):
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device=DEV).to(torch.int32)


class _Sources:
    """Background sources, each with a fixed set of peers: peer u of all sources' peers."""

    def __init__(self, g, n, s=1.1, cap=500):
        c = torch.arange(1, cap + 1, device=DEV, dtype=torch.float64)
        cdf = torch.cumsum(c.pow(-s).cpu(), 0).to(DEV)
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * cdf[-1]
        counts = torch.searchsorted(cdf, u, right=True).clamp_(max=cap - 1) + 1
        self.ends = torch.cumsum(counts, 0)
        self.total = int(self.ends[-1])
        self.ips = _ips(g, n)

    def pairs(self, g, n):
        u = torch.randint(0, self.total, (n,), generator=g, device=DEV)
        src = self.ips[torch.searchsorted(self.ends, u, right=True)]
        z = u * -7046029254386353131 + 0x1234567   # the peer's address: a mixed peer number
        z = (z ^ ((z >> 30) & 0x3FFFFFFFF)) * -4658895280553007687
        z = z ^ ((z >> 27) & 0x1FFFFFFFFF)
        return src, z.to(torch.int32)


def _with_planted(g, srcs, n, ips, lo, hi):
    """n pairs in random order: each planted host with U[lo, hi] random peers (at most half of the
    pairs in all), the rest background."""
    cards = torch.randint(lo, hi + 1, (len(ips),), generator=g, device=DEV)
    psrc = torch.repeat_interleave(ips, cards)[: n // 2]
    bsrc, bdst = srcs.pairs(g, n - len(psrc))
    src = torch.cat([psrc, bsrc])
    dst = torch.cat([_ips(g, len(psrc)), bdst])
    perm = torch.randperm(n, generator=g, device=DEV)
    return torch.stack([src[perm], dst[perm]], dim=1).contiguous()


def _inputs(case, seed):
    """One [n, 2] int32 tensor per router (or per slice of the sliding window)."""
    parts = case.get("routers", case.get("slices", 1))
    g = _gen(seed, 0)
    srcs = _Sources(g, case["sources"])
    ips = _ips(g, case["planted"])
    if case["kind"] == "routers":   # the planted hosts' peers are split over the routers
        lo, hi = max(1, case["plo"] // parts), max(2, case["phi"] // parts)
    else:
        lo, hi = case["plo"], case["phi"]
    return [_with_planted(_gen(seed, 1, k), srcs, case["n"], ips, lo, hi) for k in range(parts)]


def _params(case):
    """The hash parameters are the same for every seed, as a deployment's would be."""
    rng = random.Random(0x51A7E5EED)
    lr = case["lr"]
    mul = [rng.getrandbits(64) | 1 for _ in range(3 + lr)]
    add = [rng.getrandbits(64) for _ in range(3 + lr)]
    window = case["slices"] if case["kind"] == "sliding" else 0
    return spd.make_params(THETA, case["r"], SR, A, LOG2K, lr, case["log2lc"], mul, add, window_slices=window,
                           sliding_counter=case.get("counter", 0))


class _State:
    pass


def _tables(case):
    n = case["routers"] if case["kind"] == "serving" else 2 if case["kind"] == "both" else 1
    return [np.zeros((256 + 4 * case["planted"], 4), np.uint32) for _ in range(n)]


def prepare(case, seed):
    s = _State()
    s.kind, s.case = case["kind"], case
    s.tables = _tables(case)
    s.x = _inputs(case, seed)
    p = _params(case)
    if s.kind == "serving":
        s.srv = spd.Server(p, case["routers"], window_pairs=case["n"])
        # each router's window cut into batches of log-uniform size, the routers' batches interleaved
        rng = random.Random(seed)
        arrivals = []
        for r in range(case["routers"]):
            at = 0
            while at < case["n"]:
                m = min(case["n"] - at, _log_uniform(rng, 1 << 12, 1 << 22))
                arrivals.append((rng.random(), r, s.x[r][at:at + m]))
                at += m
        arrivals.sort(key=lambda a: a[0])
        s.sched = s.srv.schedule([0.0] * len(arrivals), [a[1] for a in arrivals], [a[2] for a in arrivals])
        return s
    s.det = spd.Detector(p, n_routers=2 if s.kind == "both" else case.get("routers", 1))
    if s.kind == "host":
        host = torch.empty(s.x[0].shape, dtype=torch.int32, pin_memory=True)
        host.copy_(s.x[0])
        s.x = host
    elif s.kind == "sliding":
        for k, x in enumerate(s.x):
            if k:
                s.det.slide()
            s.det.scan(0, x)
        s.at = 0   # the next pass's slice: the window is always the whole ring of slices
    return s


def _rows(s, report, k=0):
    """A report as the caller keeps it: its length and its records in a table of fixed size."""
    n, table = len(report), s.tables[k]
    m = min(n, len(table))
    table[:m] = report.view(np.uint32).reshape(-1, 4)[:m]
    table[m:] = 0
    return [n, table]


def run(s):
    if s.kind == "window":
        s.det.scan(0, s.x[0])
        return _rows(s, s.det.close_window(0))
    if s.kind == "noalloc":
        s.det.scan_noalloc(0, s.x[0])
        return _rows(s, s.det.close_window(0))
    if s.kind == "host":
        s.det.scan_host(0, s.x)
        return _rows(s, s.det.close_window(0))
    if s.kind == "both":
        s.det.scan_batches([(0, s.x[0]), (1, s.x[0], spd.BATCH_DST)])
        a, b = s.det.close_begin(0), s.det.close_begin(1)
        return [_rows(s, s.det.close_end(a)), _rows(s, s.det.close_end(b), 1)]
    if s.kind == "routers":
        s.det.scan_batches([(r, x) for r, x in enumerate(s.x)], merge=True)
        out = _rows(s, s.det.close_window(spd.GLOBAL))
        for r in range(len(s.x)):
            s.det.reset(r)
        return out
    if s.kind == "sliding":
        s.det.slide()
        s.det.scan(0, s.x[s.at])
        s.at = (s.at + 1) % len(s.x)
        return _rows(s, s.det.close_window(0))
    s.srv.replay(s.sched)
    s.srv.drain()
    done = [s.srv.next() for _ in range(s.case["routers"])]
    return [_rows(s, sp, hdr["router"]) for hdr, sp in sorted(done, key=lambda d: d[0]["router"])]


def work(case):
    """The pairs once, and per report the SEAV (bits, or the sliding window's counters) once; the
    hashes' multiply-adds as the operations."""
    p = _params(case)
    seav = spd.spd_derive(p).seav_bytes
    parts = case["routers"] if case["kind"] in ("routers", "serving") else 1
    keyed = 2 if case["kind"] == "both" else 1
    reports = case["routers"] if case["kind"] == "serving" else keyed
    per_bit = (0.125 * (16 if case["counter"] else 8)) if case["kind"] == "sliding" else 0.125
    pairs = case["n"] * parts
    return {"bytes": 8 * pairs + reports * seav * 8 * per_bit, "flops": 2.0 * pairs * keyed * (2 + case["lr"])}


# ------------------------------------------------------------------------------ exact
def _hash(x, mul, add, bits):
    """((mul * x + add) mod 2^64) >> (64 - bits) of 32-bit x held in int64."""
    sm, sa = (v - (1 << 64) if v >> 63 else v for v in (mul, add))
    h = ((x * sm + sa) >> 32) & 0xFFFFFFFF
    return h >> (32 - bits)


def _detect(p, parts):
    """The report of one window over the pairs of all parts, from the method's definitions: every host
    whose SEU weighs at least 3 (brute force over all 2^32 hosts) and whose ULDC estimate reaches theta."""
    d = spd.spd_derive(p)
    L, lr, k = 32 - p.r, p.lr, 1 << p.log2k
    isb, ibn = list(d.isb[:p.sr]), list(d.ibn[:p.sr])
    ldca = torch.zeros(lr << (p.log2lc + p.log2k), dtype=torch.bool, device=DEV)
    off = [0]
    for b in ibn:
        off.append(off[-1] + (1 << b))
    seav = torch.zeros((1 << p.r) * off[-1] * 8, dtype=torch.bool, device=DEV)

    def row_index(lp, i):
        return (((lp | (lp << L)) >> isb[i]) & ((1 << ibn[i]) - 1))

    for part in parts:
        for x in part.split(1 << 23):
            x = x.to(torch.int64) & 0xFFFFFFFF
            hip, oip = x[:, 0], x[:, 1]
            q = _hash(oip, p.hash_mul[2], p.hash_add[2], p.log2k)
            for i in range(lr):
                col = _hash(hip, p.hash_mul[3 + i], p.hash_add[3 + i], p.log2lc)
                ldca[(((i << p.log2lc) + col) << p.log2k) + q] = True
            keep = (_hash(oip, p.hash_mul[0], p.hash_add[0], 32) & ((1 << d.tau) - 1)) == 0
            hip, oip = hip[keep], oip[keep]
            b = _hash(oip, p.hash_mul[1], p.hash_add[1], 3)
            rp, lp = hip & ((1 << p.r) - 1), hip >> p.r
            for i in range(p.sr):
                seav[(rp * off[-1] + off[i] + row_index(lp, i)) * 8 + b] = True
    weights = (1 << torch.arange(8, device=DEV)).to(torch.uint8)
    se = (seav.view(-1, 8).to(torch.uint8) * weights).sum(1, dtype=torch.uint8).view(1 << p.r, off[-1])
    hot = torch.tensor([bin(v).count("1") >= 3 for v in range(256)], device=DEV)
    lps = torch.arange(1 << L, device=DEV)
    idx = [off[i] + row_index(lps, i) for i in range(p.sr)]
    cands = []
    step = max(1, (1 << 24) >> L)
    for r0 in range(0, 1 << p.r, step):
        rows = se[r0:r0 + step]
        seu = rows.index_select(1, idx[0])
        for i in range(1, p.sr):
            seu &= rows.index_select(1, idx[i])
        at = torch.nonzero(hot[seu.to(torch.int32)])
        cands.append((at[:, 1] << p.r) | (at[:, 0] + r0))
    cand = torch.sort(torch.cat(cands)).values
    ldca = ldca.view(-1, k)
    rep = []
    for c in cand.split(1 << 13):
        u = None
        for i in range(lr):
            row = ldca[(i << p.log2lc) + _hash(c, p.hash_mul[3 + i], p.hash_add[3 + i], p.log2lc)]
            u = row if u is None else u & row
        z0 = k - u.sum(1)
        est = -k * torch.log(z0.clamp(min=1).double() / k)
        ok = est >= p.theta
        rep.append(torch.stack([c, z0, torch.floor(est + 0.5).long(), (z0 == 0).long()], 1)[ok])
    out = torch.cat(rep) if rep else torch.zeros((0, 4), dtype=torch.int64)
    return out.cpu().numpy().astype(np.uint32)


def exact(case, seed):
    x = _inputs(case, seed)
    s = _State()
    s.tables = _tables(case)
    p = _params(case)
    if case["kind"] == "both":
        return [_rows(s, _detect(p, x)), _rows(s, _detect(p, [x[0].flip(1)]), 1)]
    if case["kind"] == "serving":
        return [_rows(s, _detect(p, [v]), r) for r, v in enumerate(x)]
    return _rows(s, _detect(p, x))   # routers: the union; sliding: the window is the whole ring of slices
