"""The benchmark's kernel durations and launch geometry where matching and the
final check are one kernel (no GPU)."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402

STAGE_MS = {"descriptor": 0.066, "support": 0.116, "filter": 0.025, "rows": 0.009, "mesh": 0.075,
            "raster": 0.071, "dense": 0.1295, "lrcheck": 0.0155}


def test_match_is_one_launch_up_to_its_limit():
    assert bench.match_in_one(640) and bench.match_in_one(2112) and not bench.match_in_one(2113)
    one, two = bench.launched(STAGE_MS, 640), bench.launched(STAGE_MS, 2113)
    assert abs(one["match"] - 0.145) < 1e-9 and "dense" not in one and "lrcheck" not in one
    assert two == STAGE_MS
    wg = bench.workgroups(320, 240, 64)
    assert wg["match"] == 240


def test_match_moves_the_check_as_well():
    # 32 pairs of 640x480: descriptors and priors read, both maps written, 2 views
    nbytes, ops = bench.algorithmic_work("match", 640, 480, {"dense_evals": 100}, pairs=32)
    assert nbytes == 32 * 2 * 640 * 480 * 22 and ops == 1600
    st = {"dense_evals": 32 * 3_200_000}
    roof = bench.roofline_of("match", 640, 480, st, 0.145, "k_matchnt_batch", pairs=32, workload="none")
    # 432.5 MB in 145 us
    assert roof["bound"] == "hbm" and abs(roof["achieved"] - 432.5e6 / 145e-6 / 1e9) < 1.0


def test_mesh_workgroups_follow_the_call():
    # 127 x 95 lattice points: 36 each for one frame, 384 over 32 pairs, 128 over 8
    assert bench.mesh_workgroups(640, 480, 1) == 2 * (-(-127 * 95 // 36) + 1)
    assert bench.mesh_workgroups(640, 480, 32) == 2 * (-(-127 * 95 // 384) + 1)
    assert bench.mesh_workgroups(640, 480, 8) == 2 * (-(-127 * 95 // 128) + 1)
    assert bench.mesh_workgroups(97, 61, 4) == 2 * (-(-18 * 11 // 72) + 1)
