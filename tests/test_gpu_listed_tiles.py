"""GPU parity of traffic with a popular sampled peer, bit-exact against the oracle.

One sampled peer with a few per cent of the pairs (a victim of an attack, or the scanner in the
destination-keyed direction) gives nearly every binning tile more sampled pairs than it stages.
Such tiles are read again when the SEAV's buckets are in memory, shared out among the workgroups of
the SEAV's buckets: one bucket and many, several slots of which some list nothing, a last tile that
is not full, one flow that sets the same bits over and over, the fused router merge (the global
sketch gets the bits too), the allocation-free scan, and launches in a row (each leaves the counts
of the next at zero).
"""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import (assert_same_report, assert_same_sketch, log, oracle_sketch, random_pairs, sampled_oips, set_tuning,
                      to_dev)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

P1M = st.CONFIGS["plain_1m"].params           # 128 KiB SEAV
BIG = P1M.replace(r=12, log2lc=13)            # 4 MiB SEAV


def traffic(mp, rng, n, share, flow=False):
    """n pairs, `share` of them with one sampled peer; flow: all of those from one host."""
    pairs = random_pairs(rng, n, n_hosts=max(2, n // 30))
    m = rng.random(n) < share
    pairs[m, 1] = sampled_oips(mp, 1, rng)[0]
    if flow:
        pairs[m, 0] = pairs[0, 0]
    return pairs


CASES = [   # parameters, pairs, share, one flow, launch settings
    (P1M, 300_001, 0.05, False, {}),
    (P1M, 1_000_003, 0.2, True, {}),
    (P1M, 2_049, 1.0, False, dict(direct_max_pairs=0)),
    (P1M, 400_001, 0.1, False, dict(direct_max_pairs=0, bucket_bits=12, bin_block=256, tile_pairs=2048, apply_block=256, apply_unroll=8)),
    (P1M, 400_001, 0.1, True, dict(direct_max_pairs=0, bucket_bits=20, bin_block=512, apply_block=512, apply_unroll=32)),
    (BIG, 1_500_001, 0.03, False, {}),
    (BIG, 700_001, 0.6, True, dict(region_words=1)),
    (P1M.replace(log2k=5, log2lc=2, lr=1), 50_001, 0.3, False, dict(direct_max_pairs=0)),   # buckets of 2^7 bits
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("noalloc", [False, True])
def test_window(case, noalloc):
    mp, n, share, flow, tune = CASES[case]
    rng = np.random.default_rng(901 + case)
    det = spd.Detector(spd.params_from(mp))
    try:
        if tune:
            set_tuning(det, **tune)
        for k, m in enumerate((n, n // 2 + 1, n)):   # the second window lists nothing
            pairs = traffic(mp, rng, m, 0.0 if k == 1 else share, flow)
            log(f"case listed tiles {case}, no-alloc {noalloc}, window {k}: {m} pairs")
            x = to_dev(pairs)
            if noalloc:
                det.scan_noalloc(0, x)
            else:
                det.scan(0, x)
            ref = oracle_sketch(mp, pairs)
            assert_same_sketch(det, 0, ref, f"window {k}")
            if mp is BIG:
                assert_same_report(det.close_window(0), ref.detect(), f"window {k}")
            det.reset(0)
    finally:
        det.close()


@pytest.mark.parametrize("merge", [False, True])
def test_routers(merge):
    """Routers of uneven size, one in two with a popular peer; two rounds, the second on slots that hold
    the first's bits."""
    rng = np.random.default_rng(951)
    R = 5
    det = spd.Detector(spd.params_from(BIG), n_routers=R)
    try:
        seen = [[] for _ in range(R)]
        for k in range(2):
            log(f"case listed tiles of {R} routers, merge {merge}, round {k}")
            for r in range(R):
                seen[r].append(traffic(BIG, rng, 120_001 + 90_000 * r, 0.08 if (r + k) % 2 else 0.0))
            det.scan_batches([(r, to_dev(seen[r][k])) for r in range(R)], merge=merge)
            for r in range(R):
                assert_same_sketch(det, r, oracle_sketch(BIG, np.concatenate(seen[r])), f"router {r}")
            if merge:
                assert_same_sketch(det, spd.GLOBAL, oracle_sketch(BIG, np.concatenate(sum(seen, []))), "global")
    finally:
        det.close()
