"""Scans recorded into a graph (stream capture) and replayed, bit-exact against the oracle.

A replay runs the recorded launches on whatever the pair buffer then holds, as often as the caller
likes and between eager scans of the same context: the counters of the region layout must be zero
for every one of them, whichever ran before.  The traffic has tiles with more sampled pairs than
they stage (a run of sampled destinations at tau = 1), whose list is the one counter that a launch
leaves for the next to clear.  A small scan under capture takes the kernel without scratch, and so
never allocates there.
"""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_sketch, log, oracle_sketch, overflow_traffic, random_pairs, set_tuning, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

MP = st.CONFIGS["plain_1m"].params.replace(theta=16)
N = 150_001


def traffic(rng, hosts):
    pairs, _ = overflow_traffic(MP, rng, hosts, 2200, noise=N)
    return pairs[len(pairs) - N:]


@pytest.mark.parametrize("small,warm", [(True, False), (True, True), (False, True)])
def test_replayed_scan(small, warm):
    rng = np.random.default_rng(61 + 2 * small + warm)
    det = spd.Detector(spd.params_from(MP))
    s = torch.cuda.Stream()
    try:
        if not small:
            set_tuning(det, direct_max_pairs=0)
        with torch.cuda.stream(s):
            x = to_dev(traffic(rng, 12))
            if warm:   # scratch of this size is there, and the last eager launch listed tiles
                for _ in range(12):
                    det.scan(0, x)
                    det.reset(0)
                assert det.stats.binned_launches > 0
            first = random_pairs(rng, 50)
            det.scan(0, to_dev(first))   # (recorded into a slot that holds bits: no clear in the graph)
            s.synchronize()
            log(f"case capture, small {small}, warm {warm}")
            binned = det.stats.binned_launches
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s, capture_error_mode="thread_local"):
                det.scan(0, x)
            assert (det.stats.binned_launches > binned) == (not small)
            for k, hosts in enumerate((14, 1, 20)):
                seen = [first] if k == 0 else [random_pairs(rng, 50)]
                if k:
                    det.reset(0)
                    det.scan(0, to_dev(seen[0]))
                for rep in range(3):   # replays in a row, an eager scan of the same size after the second
                    pairs = traffic(rng, hosts)
                    x.copy_(to_dev(pairs))
                    log(f"  replay {rep} of window {k}")
                    g.replay()
                    seen.append(pairs)
                    if rep == 1:
                        eager = traffic(rng, 13)
                        det.scan(0, to_dev(eager))
                        seen.append(eager)
                s.synchronize()
                assert_same_sketch(det, 0, oracle_sketch(MP, np.concatenate(seen)), f"window {k}")
    finally:
        s.synchronize()
        det.close()


def test_recorded_scratch_stays():
    """A graph holds a large scan; small scans of another geometry follow, which would have grown the
    scratch that the graph uses: they stay direct, and the replays are right."""
    mp = st.CONFIGS["plain_1m"].params.replace(r=12, log2lc=14)   # 17 MiB
    rng = np.random.default_rng(71)
    det = spd.Detector(spd.params_from(mp))
    s = torch.cuda.Stream()
    try:
        with torch.cuda.stream(s):
            pairs = random_pairs(rng, 300_001, n_hosts=10_000)
            x = to_dev(pairs)
            det.scan(0, x)
            det.reset(0)
            first = random_pairs(rng, 50)
            det.scan(0, to_dev(first))
            s.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s, capture_error_mode="thread_local"):
                det.scan(0, x)
            held = det.stats.device_bytes
            seen = [first]
            for k in range(12):
                log(f"case recorded scratch, pass {k}")
                g.replay()
                small = random_pairs(rng, 250_001, n_hosts=8_000)
                det.scan(0, to_dev(small))
                seen += [pairs, small]
                s.synchronize()
                assert_same_sketch(det, 0, oracle_sketch(mp, np.concatenate(seen)), f"pass {k}")
                pairs = random_pairs(rng, 300_001, n_hosts=10_000)
                x.copy_(to_dev(pairs))
            assert det.stats.device_bytes == held
    finally:
        s.synchronize()
        det.close()
