"""The end of window on crowded SEAs, against a brute force over every host.

Hot lists whose product is large: the two-step search of the tuples (the longest row met by those of
the other rows that agree), with single-precision and with integer digits, every LP of an SEA where the
tuples outnumber them, short rows, LPs of more than 24 bits, queues that fill up, bits and both kinds
of counters.  The sketch is the oracle's; the candidates are found from it by testing every LP of every
SEA (the definition of Section 3.2), since the oracle's own product would take minutes here.
"""
import numpy as np
import pytest

import oracle
import synth_traffic as st
from gpu_util import assert_same_report, assert_same_sketch, heavy_hosts, log, oracle_sketch, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

P1M = st.CONFIGS["plain_1m"].params.replace(theta=16, log2k=8, log2lc=14)
CASES = {   # parameters, hosts, peers of each, what some SEA's product has to be: (at least, below), longest row
    "short_rows": (P1M.replace(r=8, sr=8), 500, 30, (2_049, 8_193), (1, 16)),
    "single_digits": (P1M.replace(r=8), 2_500, 40, (2_049, 1 << 20), (16, 1 << 16)),
    "no_overlap": (P1M.replace(r=8, a=0), 3_000, 40, (8_193, 1 << 24), (5, 1 << 16)),
    "integer_digits": (P1M.replace(r=6, sr=5, a=3), 2_000, 40, (1 << 24, 1 << 26), (16, 64)),
    "lp_26_bits": (P1M.replace(r=6), 1_500, 40, (1 << 18, 1 << 26), (16, 1 << 16)),
    "every_lp": (P1M.replace(r=12, theta=8, log2lc=16), 300_000, 6, (1 << 20, 1 << 40), (16, 1 << 16)),
    "every_lp_sr3": (P1M.replace(r=12, sr=3, a=1, theta=8, log2lc=18), 700_000, 6, (1 << 20, 1 << 40), (16, 1 << 16)),
}


def products(seav, n_rp, ibn):
    weight = np.array([bin(v).count("1") for v in range(256)])
    hot = weight[seav.reshape(n_rp, -1)] >= 3
    ends = np.cumsum([1 << b for b in ibn])
    cnt = np.stack([hot[:, e - (1 << b):e].sum(1) for e, b in zip(ends, ibn)]).astype(np.float64)
    return cnt.prod(0), cnt.max(0)


def brute_force(mp, ref):
    """The report by testing every host: SEs of every row in common at least 3 bits, ULDC past theta."""
    p = spd.params_from(mp)
    d = spd.spd_derive(p)
    L, k = 32 - mp.r, 1 << mp.log2k
    seav = torch.from_numpy(ref.seav.copy()).cuda().view(1 << mp.r, -1)
    ldca = torch.from_numpy(ref.ldca.view(np.uint8).copy()).cuda().view(mp.lr << mp.log2lc, k // 8)
    lps = torch.arange(1 << L, device="cuda")
    off = np.concatenate([[0], np.cumsum([1 << b for b in d.ibn[:mp.sr]])])
    idx = [int(off[i]) + (((lps | (lps << L)) >> d.isb[i]) & ((1 << d.ibn[i]) - 1)) for i in range(mp.sr)]
    weight = torch.tensor([bin(v).count("1") for v in range(256)], device="cuda")
    mul, add = mp.hashes()
    rep = []
    for rp in range(1 << mp.r):
        seu = seav[rp][idx[0]]
        for i in range(1, mp.sr):
            seu &= seav[rp][idx[i]]
        cand = ((torch.nonzero(weight[seu.int()] >= 3)[:, 0] << mp.r) | rp)
        u = None
        for i in range(mp.lr):
            m, a = (v - (1 << 64) if v >> 63 else v for v in (mul[3 + i], add[3 + i]))
            col = (((cand * m + a) >> 32) & 0xFFFFFFFF) >> (32 - mp.log2lc)
            row = ldca[(i << mp.log2lc) + col]
            u = row if u is None else u & row
        z0 = k - weight[u.int()].sum(1)
        est = -k * torch.log(z0.clamp(min=1).double() / k)
        ok = z0 <= d.z_theta
        rep.append(torch.stack([cand, z0, torch.floor(est + 0.5).long(), (z0 == 0).long()], 1)[ok])
    out = torch.cat(rep).cpu().numpy()
    out = out[np.argsort(out[:, 0])].astype(np.uint32)
    return np.ascontiguousarray(out).view(spd.RECORD).reshape(-1)


@pytest.mark.parametrize("counter", ["bits", "at", "stamps"])
@pytest.mark.parametrize("case", list(CASES))
def test_crowded(case, counter):
    mp, hosts, peers, (lo, hi), (row_lo, row_hi) = CASES[case]
    rng = np.random.default_rng(701 + list(CASES).index(case))
    pairs, _ = heavy_hosts(rng, hosts, peers)
    ref = oracle_sketch(mp, pairs)
    d = spd.spd_derive(spd.params_from(mp))
    prod, row = products(ref.seav, 1 << mp.r, list(d.ibn[:mp.sr]))
    log(f"case crowded {case} {counter}: products up to {prod.max():.3g}, rows up to {row.max():.0f}")
    assert ((prod >= lo) & (prod < hi) & (row >= row_lo) & (row < row_hi)).any(), "no SEA of this kind"
    sliding = {} if counter == "bits" else dict(window_slices=3, sliding_counter=int(counter == "stamps"))
    det = spd.Detector(spd.params_from(mp.replace(**sliding)))
    try:
        for part in np.array_split(pairs, 3 if sliding else 1):
            if sliding:
                det.slide()
            det.scan(0, to_dev(part))
        assert_same_sketch(det, 0, ref, case)
        want = brute_force(mp, ref)
        assert len(want) > 100
        assert_same_report(det.close_window(0, cap=1 << 22), want, f"{case} {counter}")
    finally:
        det.close()
