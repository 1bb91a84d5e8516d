"""CPU checks of figures that the benchmark states."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_bytes_of_a_launch_are_one_read_and_one_write_of_the_lattice():
    import bench

    # whatever the number of sweeps in it: 4096^2 bits 2 x 2 MiB, 400^2 bytes 2 x 160000
    big = bench.hbm_fields(4096 * 4096, bench.BYTES_PER_SITE_BITS, 28e-6)
    assert big["algorithmic_bytes_per_launch"] == 2 * 4096 * 4096 // 8 < bench.PROFILED_TRAFFIC["bytes_per_launch"]
    assert big["hbm_achieved_GBps"] == round(4194304 / 28e-6 / 1e9, 1)
    small = bench.hbm_fields(400 * 400, bench.BYTES_PER_SITE_INT8, 12e-6)
    assert small["algorithmic_bytes_per_launch"] == 2 * 400 * 400 < bench.GRID_PROFILED_TRAFFIC["plain_bytes_per_launch"]
