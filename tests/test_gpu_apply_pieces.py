"""GPU parity of the region layout's apply phase, bit-exact against the oracle.

Buckets smaller than one 16-byte load per lane and buckets of several rounds of such loads, pieces of
each size, regions that end inside a piece, and buckets that already hold bits: the second and third
batch of a window are ORed into what the first one left, then the next window starts from zero.
"""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_report, assert_same_sketch, heavy_hosts, log, oracle_sketch, set_tuning, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

MP = st.CONFIGS["plain_1m"].params


@pytest.mark.parametrize("unroll", [8, 16, 32])
@pytest.mark.parametrize("bits,block", [(12, 1024), (13, 256), (17, 512), (20, 256)])
def test_batches_of_a_window(bits, block, unroll):
    rng = np.random.default_rng(1000 * bits + unroll)
    parts = [heavy_hosts(rng, 4, 1500, noise=n)[0] for n in (150_000, 63, 40_001)]
    log(f"case apply bucket_bits={bits} block={block} unroll={unroll}")
    det = spd.Detector(spd.params_from(MP))
    try:
        set_tuning(det, direct_max_pairs=0, bin_mode=2, bucket_bits=bits, apply_block=block, apply_unroll=unroll)
        for k in range(1, 4):
            det.scan(0, to_dev(parts[k - 1]))
            assert_same_sketch(det, 0, oracle_sketch(MP, np.concatenate(parts[:k])), f"after batch {k}")
        assert_same_report(det.close_window(0), oracle_sketch(MP, np.concatenate(parts)).detect(), "report")
        det.scan(0, to_dev(parts[2]))
        assert_same_sketch(det, 0, oracle_sketch(MP, parts[2]), "next window")
    finally:
        det.close()
