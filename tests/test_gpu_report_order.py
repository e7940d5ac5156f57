"""Reports of sizes on both sides of the change of sorting method, ips that differ in one byte only or
at both ends of the range: sorted by ip and bit-exact against the oracle."""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_report, log, oracle_sketch, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

MP = st.CONFIGS["plain_1m"].params.replace(theta=64)


@pytest.mark.parametrize("hosts", [1, 31, 32, 33, 300])
@pytest.mark.parametrize("byte", [0, 3])
def test_report_order(hosts, byte):
    rng = np.random.default_rng(400 + hosts)
    ips = (np.uint32(0x01020304) ^ (np.arange(hosts, dtype=np.uint32) << np.uint32(8 * byte)))   # (300: two bytes, or wraps)
    ips[-1] = 0xFFFFFFFF
    src = np.repeat(ips, 400)
    dst = rng.integers(0, 1 << 32, size=src.size, dtype=np.uint64).astype(np.uint32)
    pairs = np.stack([src, dst], axis=1)[rng.permutation(src.size)]
    log(f"case report of {hosts} hosts, ips differing in byte {byte}")
    det = spd.Detector(spd.params_from(MP))
    try:
        det.scan(0, to_dev(pairs))
        rep = det.close_window(0)
        assert np.all(np.diff(rep["ip"].astype(np.int64)) > 0)
        assert 0xFFFFFFFF in rep["ip"]
        assert_same_report(rep, oracle_sketch(MP, pairs).detect(), f"{hosts} hosts")
    finally:
        det.close()
