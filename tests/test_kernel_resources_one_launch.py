"""Register and scratch use of the kernels that do a whole step in one launch (Cholesky, triangular solves, FP32 Gram, the steps
that the problems of an uneven call share), as test_kernel_resources does for the others. The Cholesky also counts on two
workgroups per compute unit."""
import concurrent.futures as cf

import pytest

from test_kernel_resources import _hipcc, _report

HOT = {
    "11chol_kernel": "chol.hip",
    "tri_kernelILi1ELb0": "tri.hip",
    "tri_kernelILi1ELb1": "tri.hip",
    "tri_kernelILi4ELb0": "tri.hip",
    "tri_kernelILi4ELb1": "tri.hip",
    "tri_inv_kernel": "tri.hip",
    "tri_small_kernel": "tri.hip",
    "14gram_kernel_v2E": "gram.hip",
    "gram_kernel_v2_words": "gram.hip",
    "gram_kernel_fp8_grouped": "gram.hip",
    "gram_reduce_jobs_kernel": "gram.hip",
    "refine_line_grouped_kernel": "gemv.hip",
    "rowpass_prep_jobs_kernel": "gemv.hip",
    "colpass_jobs_kernel": "gemv.hip",
    "final_decide_jobs_kernel": "apply8.hip",
    "fp8_apply_jobs_kernel": "apply8.hip",
    "t_axpy_jobs_kernel": "apply8.hip",
    "tile_sums_jobs_kernel": "sr.hip",
    "project_update_jobs_kernel": "sr.hip",
}


@pytest.fixture(scope="module")
def reports():
    if _hipcc() is None:
        pytest.skip("hipcc not available")
    srcs = sorted(set(HOT.values()))
    with cf.ThreadPoolExecutor(max_workers=len(srcs)) as ex:
        return dict(zip(srcs, ex.map(_report, srcs)))


@pytest.mark.parametrize("frag", sorted(HOT))
def test_hot_kernel_does_not_spill(reports, frag):
    hits = {name: r for name, r in reports[HOT[frag]].items() if frag in name}
    assert hits, f"no kernel matching {frag} in {HOT[frag]}"
    for name, r in hits.items():
        assert r.get("ScratchSize [bytes/lane]") == "0", (name, r)
        assert r.get("VGPRs Spill") == "0", (name, r)


def test_two_workgroups_of_the_cholesky_share_a_compute_unit(reports):
    (r,) = [r for name, r in reports["chol.hip"].items() if "11chol_kernel" in name]
    assert 2 * int(r["LDS Size [bytes/block]"]) <= 160 * 1024
    assert int(r["Occupancy [waves/SIMD]"]) >= 2
