"""Scans of at most direct_max_pairs pairs: which kernel takes them, and what they may allocate.

With the limit as a new context has it, such scans move to the binned kernels where those are
faster, once their scratch would have paid for itself; a limit that the caller set is kept to
exactly, also when it is the default's value.  Every sketch is the oracle's.
"""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_report, assert_same_sketch, log, oracle_sketch, random_pairs, set_tuning, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

MP = st.CONFIGS["plain_1m"].params
N = 200_003   # about 10 us gained a scan: the scratch (50 us) pays for itself within ten


def windows(det, seed, count=10, n=N):
    """`count` windows of n pairs, each sketch and report compared; binned launches per window."""
    rng = np.random.default_rng(seed)
    binned = []
    for k in range(count):
        pairs = random_pairs(rng, n, n_hosts=n // 30)
        before = det.stats.binned_launches
        det.scan(0, to_dev(pairs))
        binned.append(det.stats.binned_launches - before)
        ref = oracle_sketch(MP, pairs)
        assert_same_sketch(det, 0, ref, f"window {k}")
        assert_same_report(det.close_window(0), ref.detect(), f"window {k}")
    return binned


def test_a_set_limit_is_kept():
    """Setting the limit to its default value is a choice too: no binned launch and no scratch; a value
    below the scan's size sends it to the binned kernels."""
    det = spd.Detector(spd.params_from(MP))
    try:
        log("case small scans: the limit set to its default")
        set_tuning(det, direct_max_pairs=1 << 18)
        held = det.stats.device_bytes
        assert windows(det, 71) == [0] * 10
        assert det.stats.device_bytes == held
        set_tuning(det, direct_max_pairs=N - 1)
        assert windows(det, 72, count=2) == [1, 1]
    finally:
        det.close()
