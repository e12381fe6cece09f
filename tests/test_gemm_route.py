"""Which GEMM kernel a product takes, on the CPU: the rule of csrc/gemm_route.hpp,
compiled by itself.  The GPU tests that mean to run one kernel state it with the
same helper."""

import pytest

from tests.gemm_cases import CASES, FEW_STAGES
from tests.gemm_routes import kernel, route


@pytest.mark.parametrize("M,N", [((1 << 31) - 1, 8), ((1 << 31) - 1, 64), (1 << 28, 32), ((1 << 28) - 31, 33),
                                 (40, (1 << 31) - 1), (1 << 24, 1 << 10)])
def test_grids_stay_below_the_launch_limit(M, N):
    """A launch has less than 2^32 threads: 512 per workgroup, 256 with the
    tiled kernel's 256 x 256 tiles."""
    name, tiles = route(M, N, (32, 0, 0))
    assert name != "direct"
    assert tiles * (256 if name == "tiled 256x256" else 512) < 1 << 32, name


def _mix(K):
    p4, p6 = round(K * 0.75 / 32) * 32, round(K * 0.1875 / 32) * 32
    return p4, p6, K - p4 - p6


D, S1, S2, S3, S4, S5, T1, T2 = ("direct", "split 32x32", "split 64x32", "split 64x64", "split 64x96", "split 64x128",
                                 "tiled 256x128", "tiled 256x256")
# us on 256 CUs, replays of a captured graph, the weights in rotation beyond the caches
MEASURED = [
    # long K at decode sizes: few 32-row tiles, each a long chain of steps
    (8, 4096, _mix(27648), {D: 16.1, S1: 26.6, S2: 33.9}),
    (24, 4096, (27648, 0, 0), {D: 15.1, S1: 21.8, S2: 28.6}),
    (32, 6144, _mix(14336), {D: 14.8, S1: 16.1, S2: 20.5}),
    (17, 6144, (14336, 0, 0), {D: 12.1, S1: 15.0, S2: 18.1}),
    (1, 4096, (0, 14336, 0), {D: 11.1, S1: 18.2, S2: 24.0}),
    # one activation tile, whole row groups: every CU streams at the memory's rate
    (16, 24411, (2560, 1280, 1280), {D: 18.1, S1: 20.6, S2: 21.1}),
    (8, 18290, (4128, 832, 3232), {D: 24.9, S1: 28.0, S2: 29.3}),
    (16, 16852, (1024, 160, 864), {D: 8.7, S1: 9.8, S2: 10.1}),
    # two activation tiles against many weight rows of few channels
    (32, 28672, (1024, 0, 0), {D: 8.4, S1: 7.2, S2: 6.7, T1: 9.3}),
    # four activation tiles: 8-bit codes and long K on the decode kernel
    (40, 10240, (0, 0, 14336), {D: 30.6, S1: 50.8, S2: 52.8, S3: 40.8, T1: 91.6}),
    (40, 6144, (0, 0, 8192), {D: 13.9, S1: 21.4, S2: 18.4, S3: 23.6, T1: 54.6}),
    (64, 6144, (0, 0, 4096), {D: 9.9, S1: 12.2, S2: 11.0, S3: 13.8, T1: 30.2}),
    (33, 6144, _mix(14336), {D: 16.7, S1: 23.7, S2: 19.3, S3: 24.3, T1: 56.4}),
    (64, 1024, (0, 14336, 0), {D: 19.3, S1: 14.7, S2: 20.9, S3: 28.0, T1: 76.4}),
    (64, 28672, _mix(4096), {D: 22.4, S1: 25.3, S2: 22.6, S3: 20.3, T1: 23.3}),
    # few steps at prefill sizes: a K-splitting tile would mostly add up zeros
    (8192, 14336, (128, 0, 0), {S2: 212, S3: 232, S4: 232, S5: 218, T1: 62.2, T2: 65.7}),
    (2048, 28672, (256, 0, 0), {S2: 126, S3: 135, S4: 127, S5: 115, T1: 41.9, T2: 41.0}),
    (1024, 28672, (0, 0, 128), {S2: 64.4, S3: 70.4, S4: 68.3, S5: 61.2, T1: 24.0, T2: 21.6}),
    (512, 6144, (1024, 0, 0), {S2: 12.3, S3: 12.5, S4: 15.4, S5: 13.3, T1: 9.2, T2: 13.9}),
    # fewer 256 x 256 tiles than CUs can still be the better choice
    (384, 28672, _mix(4096), {S2: 71.1, S3: 70.2, S4: 66.3, S5: 65.4, T1: 46.8, T2: 38.9}),
    # the K-splitting kernel's own ground
    (128, 6144, _mix(4096), {S1: 11.1, S2: 11.2, S3: 9.2, S4: 11.2, S5: 13.2, T1: 23.0}),
    (512, 4096, _mix(4096), {S2: 16.8, S3: 15.4, S4: 18.8, S5: 12.5, T1: 22.0, T2: 31.8}),
    (333, 5120, _mix(27648), {S2: 89.8, S3: 67.6, S4: 86.2, S5: 54.0, T1: 110, T2: 137}),
    (2048, 4096, _mix(4096), {S2: 54.8, S3: 59.7, S4: 51.0, S5: 44.9, T1: 24.3, T2: 32.2}),
]


@pytest.mark.parametrize("M,N,split,times", MEASURED, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_choice_is_near_the_fastest_measured(M, N, split, times):
    """Within 8 % of the fastest (the estimates scatter by 5 to 9 %)."""
    name, _ = route(M, N, split)
    assert times[name] <= 1.08 * min(times.values()), (name, times)


@pytest.mark.parametrize("name,M,N,split", CASES, ids=str)
def test_cases_reach_the_kernel_that_they_name(name, M, N, split):
    assert kernel(M, N, split) == name


@pytest.mark.parametrize("M,N,split", FEW_STAGES, ids=str)
def test_few_stages_reach_the_tiled_kernel(M, N, split):
    assert kernel(M, N, split) == ("tiled 256x256" if (M, N, split) in FEW_STAGES[-2:] else "tiled 256x128")
