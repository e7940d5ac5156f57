"""GPU parity of the launch geometry that the library chooses by itself, bit-exact against the oracle.

With the default settings a scan takes the direct or the binned kernels, a bucket size and a tile size by
the number of pairs, the sketch and whether it is empty.  Window sizes on both sides of each choice (every
tile size from 2048 to 8192 pairs on 256 compute units), every LDCA row count of the binned scan, a second
batch into a sketch that is not empty, several routers, and the allocation-free scan.
"""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_report, assert_same_sketch, log, oracle_sketch, random_pairs, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

P1M = st.CONFIGS["plain_1m"].params
BIG = P1M.replace(r=12, log2lc=15)   # 34 MiB: more than 256 buckets of 2^20 bits
CASES = [(P1M, n) for n in (1, 1_023, 30_001, 900_001, 2_000_003, 2_500_001, 3_000_007, 3_500_003, 4_100_001)]
CASES += [(BIG, n) for n in (40_001, 1_000_000, 4_200_001)]
CASES += [(P1M.replace(lr=lr), n) for lr in (1, 3, 4) for n in (500_001, 2_300_001)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_window(case):
    mp, n = CASES[case]
    rng = np.random.default_rng(401 + case)
    pairs = random_pairs(rng, n, n_hosts=max(1, n // 30))
    more = random_pairs(rng, 30_001 if case % 2 else 200_003, n_hosts=5_000)
    log(f"case geometry r={mp.r} lr={mp.lr}: {n} pairs, then {len(more)}")
    det = spd.Detector(spd.params_from(mp))
    try:
        for k in range(2):   # the second window's scan starts from a closed one
            det.scan(0, to_dev(pairs))
            ref = oracle_sketch(mp, pairs)
            assert_same_sketch(det, 0, ref, "first batch")
            det.scan(0, to_dev(more))
            ref.scan(more)
            assert_same_sketch(det, 0, ref, "second batch")
            assert_same_report(det.close_window(0), ref.detect(), "report")
    finally:
        det.close()


@pytest.mark.parametrize("n", [3_001, 60_001, 700_001])
def test_routers_and_noalloc(n):
    rng = np.random.default_rng(500 + n)
    R = 5
    parts = [random_pairs(rng, n + 1_000 * r, n_hosts=max(1, n // 30)) for r in range(R)]
    log(f"case geometry of {R} routers x {n} pairs")
    det = spd.Detector(spd.params_from(P1M), n_routers=R)
    try:
        det.scan_batches([(r, to_dev(p)) for r, p in enumerate(parts)], merge=True)
        for r in range(R):
            assert_same_sketch(det, r, oracle_sketch(P1M, parts[r]), f"router {r}")
            det.reset(r)
        assert_same_sketch(det, spd.GLOBAL, oracle_sketch(P1M, np.concatenate(parts)), "global")
        det.scan_noalloc(0, to_dev(parts[0]))
        assert_same_sketch(det, 0, oracle_sketch(P1M, parts[0]), "no-alloc")
    finally:
        det.close()
