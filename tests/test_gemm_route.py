"""Which GEMM kernel a product takes, on the CPU: the rule of csrc/gemm_route.hpp,
compiled by itself.  The GPU tests that mean to run one kernel state it with the
same helper."""

import pytest

from tests.gemm_routes import route


@pytest.mark.parametrize("M,N", [((1 << 31) - 1, 8), ((1 << 31) - 1, 64), (1 << 28, 32), ((1 << 28) - 31, 33),
                                 (40, (1 << 31) - 1), (1 << 24, 1 << 10)])
def test_grids_stay_below_the_launch_limit(M, N):
    """A launch has less than 2^32 threads: 512 per workgroup, 256 with the
    tiled kernel's 256 x 256 tiles."""
    name, tiles = route(M, N, (32, 0, 0))
    assert name != "direct"
    assert tiles * (256 if name == "tiled 256x256" else 512) < 1 << 32, name
