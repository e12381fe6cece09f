"""GPU parity of mm_calibrate (offline channel assignment, Sec. 3.1; Def. 1):
sigma and the split against the oracle on the same seeded inputs.

The channel sums are fp64 on both sides but in different orders (the oracle
adds rows in order, the kernels in fixed row chunks), so two means can differ
by a few units in the last place.  sigma is therefore compared exactly only on
inputs whose distinct means are further apart than both sides' rounding bound
(checked on the oracle's means before comparing), and likewise no mean may sit
within that bound of a threshold; exact ties (identical columns) and the
exact-threshold case use data whose sums are exact in any order."""

import functools

import numpy as np
import pytest
import torch

from oracle import mx_oracle as O
from paper_2508_02343_amd import workloads as W
from tests.calib_cases import boundary_case, f32_bits
from tests.gpu_helpers import note, to_dev_bf16

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=None)
def _b():
    from paper_2508_02343_amd import binding

    return binding


def _gpu(bits, formats=("E3M2", "E4M3"), ld_extra=0):
    x = to_dev_bf16(bits)
    if ld_extra:
        big = torch.full((x.shape[0], x.shape[1] + ld_extra), 1e4, dtype=torch.bfloat16, device="cuda")
        big[:, : x.shape[1]] = x
        x = big[:, : bits.shape[1]]
    perm, split = _b().calibrate(x, formats)
    torch.cuda.synchronize()
    return perm.cpu().numpy(), split


def _separation_ok(bits, formats):
    """True when the oracle's means are safely ordered and clear of the
    thresholds: relative gaps above 4 L 2^-53 (twice the bound on the
    rounding of an L-term sum of positive terms, on either side)."""
    L = bits.shape[0]
    tol = 4.0 * L * 2.0 ** -53
    M = O.channel_abs_mean(bits)
    s = np.sort(M)
    gaps = np.diff(s)
    ok_order = np.all((gaps == 0) | (gaps > tol * s[1:]))
    t = float(np.abs(O.bf16_bits_to_f64(bits)).max())
    fmts = (O.E2M1, O.E3M2 if formats[0] == "E3M2" else O.E2M3)
    ok_thr = all(np.all(np.abs(M - T) > tol * T) for T in (O.quantization_threshold(f, t) for f in fmts))
    return ok_order and ok_thr


def _check(bits, formats=("E3M2", "E4M3"), ctx="", ld_extra=0):
    fm = (O.E2M1, O.FORMATS[formats[0]], O.FORMATS[formats[1]])
    assert _separation_ok(bits, formats), f"{ctx}: test input has near-ties; pick another seed"
    sigma, split = O.calibrate(bits, fm)
    note(f"calibrate {ctx} L={bits.shape[0]} K={bits.shape[1]} formats={formats} split={split}")
    perm, gsplit = _gpu(bits, formats, ld_extra)
    assert gsplit == split, (ctx, gsplit, split)
    assert np.array_equal(np.sort(perm), np.arange(bits.shape[1])), f"{ctx}: not a permutation"
    if not np.array_equal(perm, sigma):
        i = int(np.argmax(perm != sigma))
        raise AssertionError(f"{ctx}: sigma differs first at {i}: gpu {perm[i]} oracle {sigma[i]}")
    return split


@pytest.mark.parametrize("L,K,seed", [(1, 32, 0), (17, 96, 1), (64, 512, 2), (300, 4096, 3), (2048, 4096, 4),
                                      (33, 14336, 5), (64, 32768, 6)])
def test_matches_oracle(L, K, seed):
    split = _check(W.calibration_bits(L, K, seed), ctx=f"seed{seed}")
    if L > 1 and K >= 512:
        assert split[1] > 0 and split[2] > 0  # the generator puts channels in every group


def test_full_calibration_sets():
    # calibration sets of the prefill layers' widths: Llama-3.1-8B (4096,
    # 14336) and Qwen2.5-32B (5120) with 2048-8192 tokens
    for L, K, seed in ((2048, 4096, 10), (4096, 14336, 11), (8192, 5120, 12)):
        _check(W.calibration_bits(L, K, seed), ctx=f"full{seed}")


@pytest.mark.parametrize("L,K", [(5, 256), (1100, 288), (70, 8160), (2100, 8192), (70, 8224), (1500, 5632), (1500, 5664),
                                 (700, 7680), (900, 7680), (70, 7712), (3000, 64), (3200, 64), (3200, 96)])
def test_means_in_the_rank_kernel(L, K):
    """Up to 5632 channels, or 7680 with at most 12 row chunks, the rank kernel forms
    the means itself (1 to 128 row chunks, a last slice of 32 channels); above, and
    at 64 channels with more than 48 chunks, they are a launch of their own;
    columns that are equal in pairs half the width apart must keep their
    order whichever workgroups compare them."""
    bits = W.calibration_bits(L, K, L + K)
    n = min(40, K // 2)
    bits[:, K // 2:K // 2 + n] = bits[:, :n]
    _check(bits, ctx="rank means")


def test_strided_rows():
    _check(W.calibration_bits(100, 1024, 20), ctx="ld+40", ld_extra=40)


@pytest.mark.parametrize("formats", [("E2M3", "E4M3"), ("E3M2", "E5M2"), ("E2M3", "E5M2")])
def test_alternative_formats(formats):
    _check(W.calibration_bits(256, 2048, 30), formats, ctx="alt")


def test_prefill_workload_activations():
    # the benchmark's own activations (outlier channels x30): G6 empty there
    w = W.LLAMA_ATTN
    _check(w.x_bits(512), ctx=w.name)


def test_exact_ties_keep_channel_order():
    rng = np.random.default_rng(40)
    L, K = 50, 256
    x = rng.standard_normal((L, K)).astype(np.float32)
    for a, c in ((3, 200), (7, 8), (100, 9), (250, 0)):
        x[:, a] = x[:, c]  # identical columns: equal sums in any one order
    bits = f32_bits(x)
    sigma, split = O.calibrate(bits)
    note("exact ties")
    perm, gsplit = _gpu(bits)
    assert np.array_equal(perm, sigma) and gsplit == split


def test_means_exactly_at_thresholds():
    bits = f32_bits(boundary_case())
    note("threshold boundary")
    perm, split = _gpu(bits)
    assert split == (32, 32, 32)
    assert np.array_equal(perm, O.calibrate(bits)[0])


def test_all_zero_and_constant_inputs():
    note("all zero")
    perm, split = _gpu(np.zeros((9, 160), np.uint16))
    assert split == (160, 0, 0) and np.array_equal(perm, np.arange(160))
    note("constant")
    bits = f32_bits(np.full((5, 96), -3.0, np.float32))
    perm, split = _gpu(bits)
    assert (perm.tolist(), split) == (np.arange(96).tolist(), O.calibrate(bits)[1])


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_non_finite_input_is_reported(bad):
    x = np.ones((8, 64), np.float32)
    x[5, 17] = bad
    note(f"non-finite {bad}")
    perm, split = _b().calibrate_async(to_dev_bf16(f32_bits(x)))
    torch.cuda.synchronize()
    assert split.cpu().tolist() == [-1, -1, -1]
    assert np.array_equal(perm.cpu().numpy(), np.arange(64))
    with pytest.raises(ValueError):
        _b().calibrate(to_dev_bf16(f32_bits(x)))


def test_repeatable_and_workspace_reuse():
    b = _b()
    x1 = to_dev_bf16(W.calibration_bits(700, 2048, 50))
    x2 = to_dev_bf16(W.calibration_bits(90, 1024, 51))
    ws = torch.empty(b.calibrate_workspace_size(700, 2048), dtype=torch.uint8, device="cuda")
    note("workspace reuse")
    p1, s1 = b.calibrate_async(x1, workspace=ws)
    p1 = p1.clone()
    s1 = s1.clone()
    p2, s2 = b.calibrate_async(x2, workspace=ws)  # a smaller call after it
    p3, s3 = b.calibrate_async(x1, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(p1, p3) and torch.equal(s1, s3)
    sig2, sp2 = O.calibrate(W.calibration_bits(90, 1024, 51))
    assert np.array_equal(p2.cpu().numpy(), sig2) and tuple(s2.cpu().tolist()) == sp2


def test_calibrated_layer_end_to_end():
    """calibrate -> quantize X and W with its sigma and split -> GEMM, against
    the oracle's own chain on the same inputs."""
    from tests.gpu_helpers import assert_codes_equal, assert_gemm_close, y_to_f64

    b = _b()
    L, K, N = 256, 1024, 384
    xb = W.calibration_bits(L, K, 60)
    rng = np.random.default_rng(61)
    wb = f32_bits((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
    sigma, split = O.calibrate(xb)
    note(f"end to end split={split}")
    x = to_dev_bf16(xb)
    perm, gsplit = b.calibrate(x)
    assert gsplit == split
    qa = b.quantize_act(x, perm, gsplit)
    qw = b.quantize_weight(to_dev_bf16(wb), perm, gsplit)
    y = b.gemm(qa, qw)
    torch.cuda.synchronize()
    ra, rw = O.quantize_mixed(xb, sigma, split), O.quantize_mixed(wb, sigma, split)
    assert_codes_equal(qa, ra, ctx="X")
    assert_gemm_close(y_to_f64(y), O.gemm_mixed(ra, rw), ctx="Y")


def test_subnormal_channels_are_not_flushed():
    from tests.calib_cases import subnormal_case

    bits = subnormal_case()
    note("subnormal channels")
    perm, split = _gpu(bits)
    sigma, want = O.calibrate(bits)
    assert np.array_equal(perm, sigma) and split == want
