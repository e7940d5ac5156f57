"""GPU parity of the end of a sliding window, both kinds of counters, bit-exact against the oracle.

SEAs that are no whole number of 32-counter words (their last word is read from the SEA's last four
bytes), LDCA rows of less than a word per lane up to more than one round of the filter, and one to
three rows, so that candidates end at the first row or go on to others; active and expired slices.
"""
import numpy as np
import pytest

import oracle
import synth_traffic as st
from gpu_util import assert_same_report, heavy_hosts, log, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

P1M = st.CONFIGS["plain_1m"].params
K = 5
CASES = {   # parameters, isb, ibn, noise pairs per slice
    "two_cell_row": (P1M.replace(r=12, sr=3, log2lc=8, theta=64, window_slices=K), [0, 0, 9], [1, 10, 11], 5_000),
    "one_row": (P1M.replace(r=8, lr=1, log2lc=7, log2k=8, theta=64, window_slices=K), None, None, 3_000),
    "three_rows": (P1M.replace(r=8, lr=3, log2lc=8, log2k=10, theta=64, window_slices=K), None, None, 20_000),
    "two_rounds": (P1M.replace(r=8, log2lc=6, log2k=13, theta=128, window_slices=K), None, None, 8_000),
}


@pytest.mark.parametrize("counter", [0, 1])
@pytest.mark.parametrize("case", list(CASES))
def test_sliding_close(case, counter):
    mp, isb, ibn, noise = CASES[case]
    rng = np.random.default_rng(500 + list(CASES).index(case))
    det = spd.Detector(spd.params_from(mp.replace(sliding_counter=counter), isb, ibn))
    sl = oracle.SlidingSketch(oracle.params(mp.replace(window_slices=0), isb, ibn), K)
    try:
        log(f"case sliding close {case} counter={counter}")
        seen = 0
        for t in range(K + 4):
            if t:
                det.slide()
            pairs, _ = heavy_hosts(rng, 4 if t < 3 else 1, 400, noise=noise)
            det.scan(0, to_dev(pairs))
            sl.scan_slice(pairs, t)
            want = sl.bit_view(t).detect()
            assert_same_report(det.close_window(0), want, f"{case}, slice {t}")
            seen += len(want)
        assert seen >= 4 * (K + 4)
    finally:
        det.close()
