"""Rules that the host applies for the kernels, on the CPU: where a buffer over rows of S ends."""
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
