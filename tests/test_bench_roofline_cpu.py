"""The benchmark's roofline: the march kernels' own loads are served by the L1 and
the L2, so as a share of a peak they have to be held against what those return.
Counts and times of the benchmark step (4096 x 8^3 FP32, 4 views of 1024^2)."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

COUNTS = {"ray_samples": 203122296, "prim_samples": 828990301, "fwd_cells": 839102802, "fwd_pair_intervals": 28850784,
          "fwd_pair_rays": 28850784, "bwd_pairs_visited": 31250110, "bwd_pairs_replayed": 25683702,
          "bwd_cell_runs": 161978350, "bwd_grad_flush": 14730165}


def test_shares_of_a_peak_are_below_one():
    r = bench.kernel_report({"lc": COUNTS, "fwd_ms": 7.401, "bwd_ms": 4.143}, "f32", 4 * 1024 * 1024, True)
    for k in (bench.KERN_FWD, bench.KERN_BWD):
        assert 0.0 < r[k]["frac"] < 1.0, (k, r[k])
