"""GPU parity of segments that do not fit their region, bit-exact against the oracle.

In the region layout of the binned scan a tile's words past a region's capacity go to the tile's
part of a spill array and are listed as one segment of their bucket, which the apply phase reads
after the bucket's regions.  The traffic here makes such segments: hosts that send a large share of
a window's pairs (a scan attack), a window of one host, and regions of one word.  Segments longer
than one wavefront's 64 words, buckets with more segments than the wavefronts take at a time, a
partial last chunk, several slots, the fused router merge, and windows in a row (a launch leaves its
counters zero for the next).
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
CASES = {   # pairs, hosts, their share of the pairs, launch settings
    "one_host": (300_001, 1, 1.0, {}),
    "attack": (1_200_007, 4, 0.5, {}),
    "attack_dst_512": (400_003, 3, 0.4, dict(bin_block=512, apply_block=512, apply_unroll=32)),
    "every_word": (700_001, 2, 0.1, dict(region_words=1, tile_pairs=2048, bin_block=256, apply_block=256, apply_unroll=8)),
    "every_word_small_buckets": (90_001, 2, 0.1, dict(region_words=1, tile_pairs=2048, bucket_bits=14, bin_block=512)),
}


def traffic(rng, n, hosts, share):
    m = int(n * share)
    pairs = random_pairs(rng, n, n_hosts=max(2, n // 40))
    ips = st.distinct_ips(rng, hosts)
    pairs[:m, 0] = ips[rng.integers(0, hosts, size=m)]
    return pairs[rng.permutation(n)]


@pytest.mark.parametrize("case", list(CASES))
def test_segments(case):
    n, hosts, share, tune = CASES[case]
    rng = np.random.default_rng(101 + list(CASES).index(case))
    dst = "dst" in case
    det = spd.Detector(spd.params_from(MP))
    try:
        set_tuning(det, direct_max_pairs=0, bin_mode=2, **tune)
        for k, m in enumerate((n, n // 3)):
            pairs = traffic(rng, m, hosts, share)
            log(f"case segments {case}, window {k}: {m} pairs")
            x = to_dev(pairs[:, ::-1] if dst else pairs)
            det.scan_batches([(0, x, spd.BATCH_DST if dst else 0)])
            ref = oracle_sketch(MP, pairs)
            assert_same_sketch(det, 0, ref, f"{case} window {k}")
            assert_same_report(det.close_window(0), ref.detect(), f"{case} window {k}")
    finally:
        det.close()


@pytest.mark.parametrize("merge", [False, True])
def test_segments_of_several_routers(merge):
    rng = np.random.default_rng(131)
    R = 3
    det = spd.Detector(spd.params_from(MP), n_routers=R)
    try:
        set_tuning(det, direct_max_pairs=0, bin_mode=2)
        for k in range(2):
            parts = [traffic(rng, 250_000 + 90_001 * r, 2, 0.5) for r in range(R)]
            log(f"case segments of {R} routers, merge {merge}, window {k}")
            det.scan_batches([(r, to_dev(p)) for r, p in enumerate(parts)], merge=merge)
            for r in range(R):
                ref = oracle_sketch(MP, parts[r])
                assert_same_sketch(det, r, ref, f"router {r}")
                assert_same_report(det.close_window(r), ref.detect(), f"router {r}")
            if merge:
                ref = oracle_sketch(MP, np.concatenate(parts))
                assert_same_sketch(det, spd.GLOBAL, ref, "global")
    finally:
        det.close()
