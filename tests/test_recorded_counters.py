"""The committed counter records of the default kernel belong to the committed
kernel: otherwise the benchmark leaves its hardware figures out."""
import bench


def test_records_are_of_these_sources():
    assert bench.recorded(bench.HWFLOPS_PROFILE, "hw_fp32_flops_per_launch") > 0, \
        "the kernel changed: take profiles/*_hwflops.md again"
    assert bench.recorded_traffic() > 0, "the kernel changed: take profiles/*_traffic.md again"
