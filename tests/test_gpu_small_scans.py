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


def detector(budget=0, n_routers=1):
    return spd.Detector(spd.params_from(MP), n_routers=n_routers, hbm_budget_bytes=budget)


def held_after(fn):
    """(device bytes of a new context, and after fn(det))."""
    det = detector()
    try:
        a = det.stats.device_bytes
        fn(det)
        return a, det.stats.device_bytes
    finally:
        det.close()


def test_scratch_is_grown_when_it_has_paid():
    """The first windows are direct, the later ones binned; a limit that is then set ends it."""
    det = detector()
    try:
        log("case small scans: direct, then binned")
        binned = windows(det, 81, count=12)
        assert binned[0] == 0 and binned[-1] == 1 and binned == sorted(binned)
        held = det.stats.device_bytes
        windows(det, 82, count=2, n=150_001)
        assert det.stats.device_bytes == held
    finally:
        det.close()


def test_a_budget_without_room_for_scratch():
    """Every window is scanned directly, within the budget and with the same result."""
    base, _ = held_after(lambda det: None)
    det = detector(budget=base + 4096)
    try:
        log("case small scans: no room for scratch")
        assert windows(det, 83, count=14) == [0] * 14
        assert det.stats.device_bytes == base
    finally:
        det.close()


def test_scratch_of_small_scans_makes_room():
    """A budget that holds the staging buffers of a host scan or the scratch of small scans, but not
    both: the host scan is accepted as if the small scans had stayed direct."""
    chunk = 500_000
    rng = np.random.default_rng(84)
    pairs = random_pairs(rng, chunk, n_hosts=9_000)
    base, after = held_after(lambda det: windows(det, 85, count=12))
    assert after > base
    tune = dict(direct_max_pairs=1 << 30)   # (the host scan's chunk direct too: only its staging is allocated)
    det = detector(budget=base + max(2 * 8 * chunk, after - base) + 4096)
    try:
        log("case small scans: their scratch makes room")
        assert windows(det, 86, count=12)[-1] == 1
        set_tuning(det, **tune)
        det.scan_host(0, pairs, chunk_pairs=chunk)
        assert_same_sketch(det, 0, oracle_sketch(MP, pairs), "host scan")
    finally:
        det.close()


def test_budgets_of_a_large_scan():
    """A scan that wants a geometry of its own under budgets from the least scratch a layout can do with
    up to what it would like: never refused, always the same sketch."""
    rng = np.random.default_rng(87)
    parts = [random_pairs(rng, 300_001 + 70_000 * r, n_hosts=9_000) for r in range(3)]
    dev = [to_dev(p) for p in parts]

    def scan(det, mode=2):
        if mode != 2:
            set_tuning(det, bin_mode=mode, direct_max_pairs=0)
        det.scan_batches([(r, x) for r, x in enumerate(dev)])

    def held(mode):
        det = detector(n_routers=3)
        try:
            scan(det, mode)
            return det.stats.device_bytes
        finally:
            det.close()

    low, high = held(1), held(2)
    for budget in sorted({low + 65_536, *(int(low + (high - low) * k / 6) for k in range(1, 7))}):
        det = detector(budget=budget, n_routers=3)
        try:
            log(f"case large scan under {budget} bytes")
            for k in range(2):
                scan(det)
                for r in range(3):
                    assert_same_sketch(det, r, oracle_sketch(MP, parts[r]), f"router {r}")
                    det.reset(r)
            assert det.stats.device_bytes <= budget
        finally:
            det.close()


def test_budget_below_the_wanted_regions():
    """A budget that holds the region layout only with less room in its regions: still that layout (no
    counting pass), with the same sketches."""
    rng = np.random.default_rng(88)
    pairs = random_pairs(rng, 4_000_001, n_hosts=60_000)
    x = to_dev(pairs)
    ref = oracle_sketch(MP, pairs)
    base, high = held_after(lambda det: det.scan(0, x))
    det = detector(budget=base + int(0.93 * (high - base)))
    try:
        log("case regions with less room")
        for k in range(2):
            det.profile_enable(True)
            det.scan(0, x)
            prof = det.profile()
            det.profile_enable(False)
            assert prof["count"][0] == 0 and prof["bin"][0] == 1
            assert_same_sketch(det, 0, ref, f"window {k}")
            det.reset(0)
    finally:
        det.close()


@pytest.mark.parametrize("budget_mib,group,at_least", [(512, 16 << 20, 81), (256, 1 << 20, 11), (1536, 64 << 20, 44)])
def test_server_slots_under_a_budget(budget_mib, group, at_least):
    """A tight budget keeps the slots it has always held for routers that could use them all."""
    srv = spd.Server(spd.params_from(MP), 4_000, hbm_budget_bytes=budget_mib << 20, max_group_pairs=group)
    try:
        log(f"case server slots: {budget_mib} MiB, groups of {group} pairs: {srv.stats['slots']}")
        assert srv.stats["slots"] >= at_least
    finally:
        srv.close()


@pytest.mark.parametrize("room", [4_096, 40_000, 400_000])
def test_many_batches_and_later_allocations(room):
    """Small scans of one and of twenty batches in turn, then a large scan, under a budget that holds the
    scratch of the small ones and a little more: nothing is refused that a direct scan would take, and no
    allocation of a call takes the scratch away from under it."""
    rng = np.random.default_rng(89)
    base, after = held_after(lambda det: windows(det, 90, count=12))
    big = random_pairs(rng, 700_001, n_hosts=20_000)
    _, low = held_after(lambda det: (set_tuning(det, bin_mode=1, direct_max_pairs=0), det.scan_batches(
        [(0, q) for q in to_dev(big).split(40_000)])))
    det = detector(budget=max(after + room, low + room), n_routers=1)
    try:
        log(f"case small scans of many batches, {room} bytes beside their scratch")
        for k in range(14):
            pairs = random_pairs(rng, N, n_hosts=N // 30)
            x = to_dev(pairs)
            det.scan_batches([(0, q) for q in x.split(N if k % 2 else N // 20)])
            assert_same_sketch(det, 0, oracle_sketch(MP, pairs), f"window {k}")
            det.reset(0)
        for k in range(2):
            det.scan_batches([(0, q) for q in to_dev(big).split(40_000)])
            assert_same_sketch(det, 0, oracle_sketch(MP, big), f"large window {k}")
            det.reset(0)
            windows(det, 91 + k, count=2)
    finally:
        det.close()
