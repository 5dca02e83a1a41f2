"""The GEMM kernel chosen for a size, without a GPU (256 CUs are assumed there):
the GPU cases run the kernel they are listed under, and sizes whose kernels were
timed go to the fastest or, within the estimate's error, next to it.  And the sources a call's
counters are tied to."""
import os
import re

import pytest

import bench
import test_gpu_ksplit as K
from paper_2507_23035_amd import build, oasis


def route(n, d_in, d_out):
    if not os.path.exists(oasis.LIB_PATH):
        build.build()
    return oasis.load().oasis_gemm_route(n, d_in, d_out)


@pytest.mark.parametrize("n,d_in,d_out,seed,kernel", K.CASES)
def test_cases_run_the_kernel_they_name(n, d_in, d_out, seed, kernel):
    assert route(n, d_in, d_out) == kernel


# us, many-token kernel / 32 x 32 / 64 x 64 / 128 x 64 / 128 x 128 (0: not built)
TIMED = [
    (2048, 520, 4096, (21.3, 55.4, 33.3, 30.3, 0)),
    (1000, 520, 8100, (22.3, 56.1, 33.4, 30.2, 0)),
    (2500, 1032, 20000, (152.3, 399.1, 224.8, 202.4, 0)),
    (2048, 1032, 4096, (29.0, 69.1, 40.7, 36.4, 0)),
    (1500, 1544, 6000, (56.8, 90.5, 53.3, 50.0, 0)),
    (1500, 5000, 6000, (139.5, 179.6, 120.7, 119.4, 0)),
    (800, 4104, 3001, (65.4, 46.3, 37.7, 40.4, 0)),
    (100, 8200, 4000, (91.2, 19.6, 21.6, 32.1, 0)),
    (1500, 1024, 6000, (32.5, 70.4, 40.8, 40.2, 40.2)),
    (1100, 1024, 5000, (22.9, 45.6, 28.4, 25.8, 27.6)),
    (3500, 2048, 3000, (56.0, 135.4, 74.0, 68.3, 61.7)),
    (900, 8192, 12000, (193.0, 318.8, 208.3, 180.2, 173.0)),
    (1500, 8192, 6000, (176.6, 255.6, 165.9, 152.4, 170.2)),
]


@pytest.mark.parametrize("n,d_in,d_out,us", TIMED)
def test_timed_sizes(n, d_in, d_out, us):
    r = route(n, d_in, d_out)
    assert us[0 if r >= K.TILES else r] <= 1.09 * min(u for u in us if u)


def test_counters_are_tied_to_every_kernel_source():
    """bench.py drops counters once a source of the call's kernels has changed: each
    HIP source belongs to a call, and a listed one brings its headers along."""
    listed = set().union(*bench.KERNEL_SOURCES.values())
    assert {f for f in build.SOURCES if f.endswith(".hip")} <= listed
    for call, files in bench.KERNEL_SOURCES.items():
        for f in files:
            text = open(os.path.join(build.CSRC, f)).read()
            included = set(re.findall(r'#include "(\w+\.h)"', text)) - {"common.h", "oasis.h"}
            assert included <= set(files), (call, f)
