"""Occupancy and scratch of the kernels that test_kernel_resources.py does not list: the
wide workgroups of the build, the 1024-thread refit, the scan, the k nearest and the spread
order."""

import re

import pytest

from test_kernel_resources import HIPCC, _parse, _report

# kernel-name pattern -> (minimum waves per SIMD, maximum scratch bytes per lane, how many)
EXPECT = {
    "query.hip": {
        r"scan_kernelILb1EE": (5, 0, 1),
        r"scan_kernelILb0EE": (8, 0, 1),
        r"knn_batch_kernelILi(1|2|4|8|16)ELi2EE": (4, 0, 5),
        r"knn_batch_kernelILi(1|2|4|8|16)ELi4EE": (4, 0, 5),
        r"knn_batch_kernelILi(1|2|4|8)ELi8EE": (4, 0, 4),
        r"traverse_batch_kernelILb1ELi(1|2|4|8|16|32)ELi[45]EE": (5, 0, 12),   # five waves, as the default batches assume
        r"traverse_batch_kernelILb0ELi(1|2|4|8)ELi4EE": (6, 0, 4),
        r"traverse_lane_kernelILb1ELb0EE": (4, 256, 1),                        # the stack's deep end is an array
        r"cell_(count|deal)_kernel": (8, 0, 2),
    },
    "lbvh.hip": {
        # a 1024-thread workgroup is four waves on every SIMD, and its LDS leaves no room for a second
        r"refit_kernelILb[01]ELi1024ELi2ELi4EE": (4, 0, 2),
        r"frame_update_kernelILi1024ELi2ELi4EE": (4, 0, 1),
        r"small_sort_kernelILi[124]EE": (8, 0, 3),
        r"radix_pass_kernelILi(4|8|16)EE": (8, 0, 3),
        r"bounds_kernel": (8, 0, 1),
        r"order_subtrees_kernel": (8, 0, 1),
    },
    "sdf.hip": {
        r"face_record_kernel": (8, 0, 1),
        r"sdf_update_k_kernelILi[1248]ELb[01]EE": (4, 0, 8),
    },
    "losses.hip": {
        r"(point_mesh|chamfer)_backward_kernel": (8, 0, 2),
    },
}


@pytest.mark.skipif(HIPCC is None, reason="hipcc not installed")
def test_kernels_keep_their_occupancy():
    procs = {src: _report(src) for src in EXPECT}
    problems = []
    for src, proc in procs.items():
        text, _ = proc.communicate(timeout=600)
        assert proc.returncode == 0, text[-2000:]
        kernels = _parse(text)
        for pat, (waves, scratch, count) in EXPECT[src].items():
            hits = {k: v for k, v in kernels.items() if re.search(pat, k)}
            if len(hits) != count:
                problems.append(f"{src}: {len(hits)} kernels match {pat}, not {count}")
            for name, r in hits.items():
                if r.get("waves", 0) < waves or r.get("scratch", 1 << 30) > scratch:
                    problems.append(f"{name}: {r} (want >= {waves} waves/SIMD, <= {scratch} B scratch)")
    assert not problems, "\n".join(problems)
