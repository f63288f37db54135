"""bench.py's figures of single kernels (no GPU needed): its roofline names a
kernel that the steps run, and every counter-summary entry it may read belongs to
kernel sources that are there."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    sys.path.insert(0, ROOT)
    try:
        import bench as b
    finally:
        sys.path.remove(ROOT)
    return b


@pytest.mark.parametrize("line_x", [False, True])
@pytest.mark.parametrize("line_y", [False, True])
def test_roofline_names_a_kernel_of_the_step(bench, line_x, line_y):
    """iga_line_solve's kernels are the step's only where it does not solve one line per lane."""
    kt = {"assemble_s1_fuel": 3e-5, "assemble_s3": 2e-5, "line_solve_x_A": 6e-5, "line_solve_y_M": 5e-5,
          "line_solve_y_cn": 4e-5}
    sched = [{"line_per_lane": line_x}, {"line_per_lane": line_y}, {}]
    roof = bench.roofline(kt, 2, 100 ** 2, 98 ** 2, 98, sched)
    assert roof["kernel"] == ("line_solve_x_A" if not line_x else "line_solve_y_M" if not line_y
                              else "assemble_s1_fuel")
    assert roof["kernel_us"].keys() == kt.keys()


def test_counter_entries_have_sources(bench):
    for family in bench.KERNEL_FAMILY.values():
        for entry in family:
            for f in bench.SOURCES[entry.split("<")[0]]:
                assert os.path.exists(os.path.join(ROOT, "paper_2604_19370_amd", "csrc", f)), f
