"""The serving loop's closes of one scan group, in one launch: bit-exact against the oracle.

More windows than one launch names (32), windows of very different sizes beside each other, windows
without any pair between them (their slots are not read), every workgroup size of the kernel, and row
counts it treats apart (four, and others); each slot is used for a second window afterwards.
"""
import numpy as np
import pytest

import synth_traffic as st
from gpu_util import assert_same_report, heavy_hosts, log, oracle_sketch, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1901_07306_amd as spd  # noqa: E402

BASE = st.CONFIGS["plain_1m"].params.replace(r=8, log2lc=10, theta=64)
CASES = {   # parameters, routers, workgroup of the close
    "40_windows": (BASE, 40, 0),
    "block_64": (BASE, 9, 64),
    "block_256_sr2": (BASE.replace(sr=2, a=2, log2lc=8), 9, 256),
}


@pytest.mark.parametrize("case", list(CASES))
def test_windows_closed_together(case):
    mp, R, block = CASES[case]
    rng = np.random.default_rng(301 + list(CASES).index(case))
    sizes = rng.integers(0, 60_000, size=2 * R)
    sizes[rng.permutation(2 * R)[: R // 3]] = 0      # no pairs at all: closed by request only
    windows = []
    for n in sizes:
        windows.append(heavy_hosts(rng, 4, 400, noise=int(n))[0] if n else np.zeros((0, 2), np.uint32))
    log(f"case {case}: {R} routers, two windows each of up to 60000 pairs")
    tuning = None
    if block:
        det = spd.Detector(spd.params_from(mp))
        tuning = det.tuning
        det.close()
        tuning.close_block = block
    srv = spd.Server(spd.params_from(mp), n_routers=R, max_slots=R, hbm_budget_bytes=512 << 20, tuning=tuning)
    try:
        for k, pairs in enumerate(windows):
            srv.submit(k % R, to_dev(pairs) if len(pairs) else torch.empty((0, 2), dtype=torch.int32, device="cuda"),
                       close=True)
        srv.drain()
        got = {}
        for _ in windows:
            res = srv.next(timeout_ms=20000)
            assert res is not None, "a window never finished"
            hdr, sp = res
            got[(hdr["router"], hdr["window"])] = (hdr["pairs"], sp)
        for k, pairs in enumerate(windows):
            n, sp = got[(k % R, k // R)]
            assert n == len(pairs)
            assert_same_report(sp, oracle_sketch(mp, pairs).detect(), f"{case}, router {k % R} window {k // R}")
    finally:
        srv.close()
