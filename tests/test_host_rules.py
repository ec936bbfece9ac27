"""Rules that the host applies for the kernels and its launches, on the CPU."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_17556_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("rules") / "rules.so")
    cmd = [hipcc, "-O1", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950", "-x", "hip", "-I", os.path.join(ROOT, "include"),
           "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           os.path.join(ROOT, "tests", "host_rules.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    return ctypes.CDLL(out)


def words(rules, row0, rows, col0, lane_rows, lane_cols, n, m, lds):
    """The floats of S that one load of a wave touches, as offsets from S: lane l reads 4 words from row row0 + lane_rows[l],
    column col0 + lane_cols[l], as far as they lie inside the buffer's records."""
    rec = rules.rules_row_records(rows, lds, m - col0) // 4
    at = (lane_rows * lds + lane_cols)[:, None] + np.arange(4)[None, :]
    return row0 * lds + col0 + at[at < rec]


@pytest.mark.parametrize("n,m,lds", [(1, 33, 33), (1, 17, 100), (8, 40, 41), (9, 31, 64), (17, 127, 1000), (16, 128, 128),
                                     (33, 129, 131), (40, 300, 1023)])
def test_row_passes_stay_inside_S(rules, n, m, lds):
    """S is (n - 1) lds + m floats: no load of the whole-line refinement (8 rows, 32 columns) or of the multi-vector row pass
    (16 rows, steps of 128 columns) touches a float behind them, and together they touch every element."""
    end = (n - 1) * lds + m
    lane = np.arange(64)
    for rows_at_once, width, pieces in [
        (8, 32, [(lane >> 3, 4 * (lane & 7))]),
        (16, 128, [(lane & 15, 16 * u + 4 * (lane >> 4)) for u in range(8)]),
    ]:
        seen = np.zeros(end, bool)
        for r0 in range(0, n + rows_at_once, rows_at_once):
            rows = max(0, min(rows_at_once, n - r0))
            for c0 in range(0, m, width):
                for lr, lc in pieces:
                    w = words(rules, r0 if rows else 0, rows, c0, lr, lc, n, m, lds)
                    assert w.size == 0 or w.max() < end, (r0, c0)
                    seen[w] = True
        inside = np.arange(end) % lds < m
        assert seen[inside].all()


def base_slices(n, m):
    """The slice count that fills 256 compute units best with at least 2048 columns a slice: a multiple of 8."""
    ntri = (n + 255) // 256 * ((n + 255) // 256 + 1) // 2
    best, score = 1, -1.0
    for q in range(1, max(1, min(64, m // (8 * 2048))) + 1):
        rounds = (8 * q * ntri + 255) // 256
        s = 8 * q * ntri / (rounds * 256) * (1.0 if rounds >= 4 else 0.5 + 0.125 * rounds)
        if s > score + 1e-9:
            best, score = q, s
    return 8 * best


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("aligned", [1, 0])
def test_gram_slices_are_no_longer_than_the_base_plans(rules, prec, aligned):
    """A slice is summed in FP32 and slices are added in FP64, so no plan may take longer slices than the base plan."""
    ns, ks = ctypes.c_int64(), ctypes.c_int64()
    L = [ctypes.c_int64] * 3 + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int64)] * 2
    rules.rules_gram_plan.argtypes = L
    step = {0: 32, 1: 32, 2: 64}[prec]
    for n in (1, 32, 250, 257, 520, 1000, 1500, 2048, 3001, 4096, 8192):
        for m in (40, 1000, 10_000, 40_000, 99_999, 250_000, 1_000_000, 4_000_000):
            if prec == 2 and not aligned:
                continue
            rules.rules_gram_plan(n, m, m, prec, aligned, 0, -1, ns, ks)
            cap = {0: m, 1: (m + 63) // 64 * 64, 2: (m + 127) // 128 * 128}[prec]
            b = base_slices(n, m)
            most = max(1, ((cap + b - 1) // b + step - 1) // step) * step
            assert ks.value <= most, (n, m, ns.value, ks.value, b, most)
            assert ns.value * ks.value >= cap and ks.value % step == 0


class Fake:
    """A context's workspace on a device of `capacity` bytes."""

    def __init__(self, rules, capacity):
        self.r = rules
        rules.rules_ws_new.restype = ctypes.c_void_p
        rules.rules_ws_new.argtypes = [ctypes.c_size_t]
        rules.rules_ws_set.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
        rules.rules_ws_levels.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t), ctypes.c_int, ctypes.c_int]
        rules.rules_ws_counts.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_int64)]
        rules.rules_ws_delete.argtypes = [ctypes.c_void_p]
        self.h = rules.rules_ws_new(capacity)

    def set(self, capacity, frozen=False):
        self.r.rules_ws_set(self.h, capacity, frozen)

    def levels(self, *need, can_grow=True):
        return self.r.rules_ws_levels(self.h, (ctypes.c_size_t * len(need))(*need), len(need), can_grow)

    def counts(self):
        out = (ctypes.c_int64 * 5)()
        self.r.rules_ws_counts(self.h, out)
        return list(out)

    def __del__(self):
        self.r.rules_ws_delete(self.h)


def test_workspace_at_the_limit_costs_one_attempt(rules):
    """A preferred layout that does not fit is tried once: later calls neither allocate, free nor synchronise."""
    f = Fake(rules, 50)
    assert f.levels(60, 45, 40) == 1
    assert f.levels(70, 55, 45) == 2   # 55 may fit where 60 did not
    held = f.counts()
    assert held[0] == 45
    for _ in range(5):
        assert f.levels(60, 45, 40) == 1
        assert f.levels(70, 55, 45) == 2
    assert f.counts() == held
    f.set(130)   # the program gave memory back
    assert f.levels(60, 45, 40) == 0


def test_workspace_stays_when_the_smaller_layout_has_room(rules):
    f = Fake(rules, 90)
    assert f.levels(50) == 0
    assert f.levels(95, 45) == 1
    assert f.counts()[0] == 50 and f.counts()[3] == 0   # (and with it a captured sequence of launches)


def test_workspace_grows_in_place(rules):
    f = Fake(rules, 100)
    assert f.levels(50) == 0
    assert f.levels(80, 40) == 0        # beside it there is no room
    assert f.levels(101, 100) == 1      # the last resort has to grow too
    assert f.levels(101, 101) == -1


def test_workspace_held_by_a_capture(rules):
    f = Fake(rules, 1000)
    assert f.levels(50) == 0
    f.set(1000, frozen=True)
    assert f.levels(60, 50, 40) == 1 and f.levels(70, 60) == -1
    assert f.counts()[1] == 1 and f.counts()[0] == 50
    f.set(1000)
    assert f.levels(60, 50, 40, can_grow=False) == 1 and f.levels(70, 60, can_grow=False) == -1
    assert f.counts()[1] == 1


@pytest.mark.parametrize("shapes,alone", [
    ([(64, 1 << 21)], []),
    ([(64, 1 << 21), (4096, 8192)], [1]),              # 8 workgroups would walk 4096 rows behind a short launch
    ([(4096, 8192), (64, 1 << 21), (3000, 4096)], [0, 2]),
    ([(512, 8192), (64, 1 << 21)], []),
    ([(64, 1 << 21), (1024, 262144), (300, 9000)], []),
    ([(1024, 65536)] * 40, []),
    ([(64, 32768)] * 30, list(range(30))),             # too few column blocks to fill the device
    ([(4096, 8192), (64, 2040 * 1024)], [0, 1]),       # the first alone, too few left
])
def test_column_passes_that_share_a_launch(rules, shapes, alone):
    k = len(shapes)
    n, m = ((ctypes.c_int64 * k)(*v) for v in zip(*shapes))
    out = (ctypes.c_int * k)()
    took = list(out[:rules.rules_colpass_together(n, m, k, out)])
    assert sorted(set(range(k)) - set(took)) == alone
    assert [shapes[i][0] for i in took] == sorted((shapes[i][0] for i in took), reverse=True)


def test_tuner_reaches_the_built_in_plan(rules):
    """The candidates go up to at least half the built-in plan's slices (512 is the most that a tuning table can hold), so that
    tuning a context does not cost it the plan it had."""
    ns, ks, q = ctypes.c_int64(), ctypes.c_int64(), (ctypes.c_int * 16)()
    rules.rules_gram_plan.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int64)] * 2
    rules.rules_gram_candidates.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(ctypes.c_int)]
    for n in (8, 64, 256, 300, 520, 1000, 1500, 2048, 4096, 8192):
        for m in (1000, 10_000, 40_000, 100_000, 250_000, 1_000_000):
            got = list(q[:rules.rules_gram_candidates(n, m, q)])
            assert got[0] == 1 and got == sorted(got) and got[-1] <= 64
            for prec in (0, 1, 2):
                rules.rules_gram_plan(n, m, m, prec, 1, 0, -1, ns, ks)
                assert 8 * got[-1] >= min(ns.value, 512) / 2, (n, m, prec, got, ns.value)
