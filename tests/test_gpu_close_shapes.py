"""GPU parity of the end of window over the shapes of an SEA, bit-exact against the oracle.

Rows of two cells (an SEA that is no whole number of words), every row count the kernel treats apart
(four, and others), hot lists longer than a wavefront, tuple counts on both sides of the limits (all
parts enumerate; single-precision digits; integer digits), more records than travel with the counts,
collected by both closes, and AT windows around half the code period.
"""
import numpy as np
import pytest

import oracle
import synth_traffic as st
from gpu_util import assert_same_report, assert_same_sketch, heavy_hosts, log, oracle_sketch, set_tuning, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

P1M = st.CONFIGS["plain_1m"].params
CASES = {   # parameters, isb, ibn, hosts, peers of each, other pairs
    "two_cell_row": (P1M.replace(r=12, sr=3, log2lc=8, theta=64), [0, 0, 9], [1, 10, 11], 30, 400, 20_000),
    "sr8": (P1M.replace(r=8, sr=8, a=2, log2lc=8, theta=64), None, None, 20, 400, 5_000),
    "sr2": (P1M.replace(r=10, sr=2, a=2, log2lc=8, theta=64), None, None, 20, 400, 5_000),
    "tuples_1e4": (P1M.replace(theta=16, log2k=8), None, None, 640, 40, 0),
    "tuples_1e6": (P1M.replace(r=3, theta=16, log2k=8), None, None, 330, 40, 0),
    "records": (P1M.replace(r=12, theta=16, log2k=8), None, None, 6_000, 60, 0),
}


@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("case", list(CASES))
def test_close_shapes(case, block):
    mp, isb, ibn, hosts, peers, noise = CASES[case]
    rng = np.random.default_rng(211 + list(CASES).index(case))
    pairs, _ = heavy_hosts(rng, hosts, peers, noise=noise)
    log(f"case close {case} block={block}: {len(pairs)} pairs")
    ref = oracle_sketch(mp, pairs, isb, ibn)
    want = ref.detect()
    assert len(want) >= hosts // 2
    det = spd.Detector(spd.params_from(mp, isb, ibn))
    try:
        set_tuning(det, close_block=block)
        x = to_dev(pairs)
        det.scan(0, x)
        assert_same_sketch(det, 0, ref, case)
        assert_same_report(det.close_window(0), want, f"{case}, blocking close")
        det.scan(0, x)
        ticket = det.close_begin(0)
        det.scan(0, x[: len(x) // 2])
        assert_same_report(det.close_end(ticket), want, f"{case}, two-part close")
    finally:
        det.close()


@pytest.mark.parametrize("K", [127, 128, 129])
def test_at_window_around_half_the_period(K):
    """Slices 0 .. 2 K + 3 of small traffic whose hosts go silent halfway: counters of every age up to
    and past K, reports against the oracle at the window's edges."""
    mp = P1M.replace(r=8, log2lc=6, log2k=8, theta=64, window_slices=K)
    rng = np.random.default_rng(300 + K)
    first, _ = heavy_hosts(rng, 6, 400)
    det = spd.Detector(spd.params_from(mp))
    sl = oracle.SlidingSketch(oracle.params(mp.replace(window_slices=0)), K)
    try:
        log(f"case AT window K={K}")
        seen = 0
        for t in range(2 * K + 4):
            if t:
                det.slide()
            pairs = first if t in (0, K // 2) else heavy_hosts(rng, 1, 120)[0]
            det.scan(0, to_dev(pairs))
            sl.scan_slice(pairs, t)
            if t in (0, K - 1, K, K + K // 2 - 1, K + K // 2, K + K // 2 + 1, 2 * K + 3):
                want = sl.bit_view(t).detect()
                assert_same_report(det.close_window(0), want, f"K={K}, slice {t}")
                seen += len(want)
        assert seen > 12
    finally:
        det.close()
