"""The serving loop's scratch is reserved at creation: groups of few and of many windows of a small
sketch, whose launches choose geometries of their own (more and smaller buckets, smaller tiles),
allocate no device memory; with a budget that leaves room for nothing else the tuning's geometry or
the direct kernel serves, with the same reports.
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

MP = st.CONFIGS["plain_1m"].params.replace(r=8, log2lc=10, theta=512)   # 9 buckets of 2^20 bits


def serve(srv, counts, rng, R):
    for k, n_win in enumerate(counts):
        windows = [heavy_hosts(rng, 3, 700, noise=int(rng.integers(20_000, 300_000) / n_win ** 0.5))[0] for _ in range(n_win)]
        x = [to_dev(w) for w in windows]
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        log(f"  group of {n_win} windows")
        order = rng.permutation(R)[:n_win]
        sched = srv.schedule([0.0] * n_win, [int(r) for r in order], x, flags=[spd.SPD_SUBMIT_CLOSE] * n_win)
        srv.replay(sched)
        srv.drain()
        for _ in range(n_win):
            hdr, sp = srv.next(timeout_ms=20000)
            w = windows[list(order).index(hdr["router"])]
            assert hdr["pairs"] == len(w)
            assert_same_report(sp, oracle_sketch(MP, w).detect(), f"group of {n_win}, router {hdr['router']}")
        # (the HIP runtime allocates for itself at a stream's first launches: not at the first group)
        assert k == 0 or torch.cuda.mem_get_info()[0] == free, f"a group of {n_win} windows allocated device memory"


@pytest.mark.parametrize("budget", [0, 1])
def test_groups(budget):
    R = 32
    rng = np.random.default_rng(611 + budget)
    p = spd.params_from(MP)
    kw = dict(max_slots=64) if not budget else dict(hbm_budget_bytes=60 << 20, max_group_pairs=1 << 18, max_group_batches=64)
    srv = spd.Server(p, R, **kw)
    try:
        log(f"case server scratch, budget {budget}, slots {srv.stats['slots']}")
        serve(srv, [1, 2, 5, 8, 17, 32, 1, 3] if not budget else [1, 5, 12, 1], rng, R)
    finally:
        srv.close()
