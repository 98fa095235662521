"""bench.py's roofline names the kernel that the headline call runs, counts its operations,
and guards that kernel's measured traffic by the source that it is built from (no GPU)."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2602_15605_amd", "csrc")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def test_headline_kernels():
    assert bench.reduction_kernel("fp32c", 6000) == ("strip_fp32c_kernel", 12)
    assert bench.reduction_kernel("fp64", 6000) == ("tile_pol_kernel", 10)
    assert bench.reduction_kernel("fp64", bench.TILE_FROM - 1) == ("strip_fp64_kernel", 12)
    assert bench.TILE_FROM == int(re.search(r"kTileMinPol = (\d+)", _source("strip_params.hpp")).group(1))


def test_traffic_is_kept_for_the_kernels_and_guarded_by_their_sources():
    guarded = {os.path.basename(p) for p in bench.KERNEL_SOURCES}
    with open(bench.TRAFFIC_PROFILE) as f:
        profile = f.read()
    for prec in ("fp32c", "fp64"):
        kernel, _ = bench.reduction_kernel(prec, 6000)
        assert "traffic_bytes_per_launch %s =" % kernel in profile
        home = [n for n in os.listdir(CSRC) if re.search(r"__global__[^;{]*\b%s\(" % kernel, _source(n))]
        assert home and set(home) <= guarded, (kernel, home)
    assert "strip_params.hpp" in guarded
