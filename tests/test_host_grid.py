"""Launch grids at the largest sizes, on the host build."""
import ctypes as C
import os

import pytest

HC_PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_03031_amd", "lib",
                       "libvc_hostcheck.so")


@pytest.fixture(scope="module")
def hc():
    if not os.path.exists(HC_PATH):
        from paper_2601_03031_amd import build as B
        B.build_hostcheck()
    return C.CDLL(HC_PATH)


@pytest.mark.parametrize("log_n", range(2, 31))
def test_a_workgroup_per_proof(hc, log_n):
    """Every proof has its workgroup of 256 threads, and no dimension 2^32 threads or more than 2^16
    workgroups beside the first."""
    xy = (C.c_uint32 * 2)()
    hc.hc_proof_grid(C.c_uint64(1 << log_n), xy)
    x, y = xy
    assert x * y == 1 << log_n and 256 * x < 1 << 32 and y < 1 << 16
    assert y == 1 or x == 1 << 16  # proof 2^16 y + x
