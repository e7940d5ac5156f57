"""The end-of-window kernel's LDS limit: a layout whose dynamic LDS fills the compute unit's exactly at
256 lanes (the kernel has static LDS too, so fewer lanes take it), against the oracle, and a layout of
unequal rows past the limit, which is refused."""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_report, heavy_hosts, log, oracle_sketch, set_tuning, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

MP = st.CONFIGS["plain_1m"].params.replace(r=8, sr=4, log2lc=8, theta=64)


@pytest.mark.parametrize("block", [64, 256])
def test_lds_filled_exactly(block):
    isb, ibn = [0, 13, 16, 4], [13, 10, 9, 8]   # 9984 SEs: 4 wavefronts x (9984 + 256) words are 160 KiB
    rng = np.random.default_rng(31)
    pairs, _ = heavy_hosts(rng, 20, 400, noise=5_000)
    det = spd.Detector(spd.params_from(MP, isb, ibn))
    try:
        set_tuning(det, close_block=block)
        log(f"case close with its LDS filled, block {block}")
        det.scan(0, to_dev(pairs))
        want = oracle_sketch(MP, pairs, isb, ibn).detect()
        assert len(want) >= 10
        assert_same_report(det.close_window(0), want, "report")
    finally:
        det.close()


def test_long_row_is_refused():
    det = spd.Detector(spd.params_from(MP.replace(r=3, sr=3), [0, 15, 20], [15, 12, 10]))
    try:
        log("case close with a row past the limit")
        det.scan(0, to_dev(heavy_hosts(np.random.default_rng(32), 2, 100)[0]))
        with pytest.raises(spd.SpdError) as e:
            det.close_window(0)
        assert e.value.status == spd.SPD_E_INVALID
    finally:
        det.close()
