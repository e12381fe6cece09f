"""GPU parity of the mixed-precision GEMM (mm_gemm) against the oracle's float64
product of the dequantised operands, within |gpu - ref| <= 2^-8 |ref| +
1e-3 rms(ref).  The quantised operands come from the HIP quantiser, whose
bytes are first checked against the oracle, so both sides multiply the same
codes."""

import functools

import numpy as np
import pytest
import torch

from oracle import mx_oracle as O
from paper_2508_02343_amd import workloads as W
from tests.gemm_cases import CASES, FEW_STAGES
from tests.gpu_helpers import assert_codes_equal, assert_gemm_close, note, to_dev_bf16, to_dev_perm, y_to_f64

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=None)
def _b():
    from paper_2508_02343_amd import binding

    return binding


def _gpu_pair(xb, wb, perm, split):
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split)
    w = b.quantize_weight(to_dev_bf16(wb), p, split)
    return a, w


def _check_full(xb, wb, perm, split, ctx):
    a, w = _gpu_pair(xb, wb, perm, split)
    y = _b().gemm(a, w)
    torch.cuda.synchronize()
    ra, rw = O.quantize_mixed(xb, perm, split), O.quantize_mixed(wb, perm, split)
    assert_codes_equal(a, ra, ctx=ctx + " A")
    assert_codes_equal(w, rw, ctx=ctx + " W")
    assert_gemm_close(y_to_f64(y), O.gemm_mixed(ra, rw), ctx=ctx)


def test_tiny_config():
    w = W.TINY
    note(w.name)
    _check_full(w.x_bits(), w.w_bits(), w.perm(), w.split, w.name)


def _rand_case(M, N, split, seed):
    K = sum(split)
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, K)).astype(np.float32)
    out = rng.choice(K, max(1, K // 64), replace=False)
    x[:, out] *= 25
    perm = np.concatenate([np.setdiff1d(np.arange(K), out), out]).astype(np.int32)
    wgt = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    return W.f32_to_bf16_bits(x), W.f32_to_bf16_bits(wgt), perm


@pytest.mark.parametrize("split", [(96, 160, 96), (352, 0, 0), (0, 352, 0), (0, 0, 352), (32, 32, 288),
                                   (128, 0, 224), (0, 64, 32)])
@pytest.mark.parametrize("M,N", [(1, 16), (5, 70), (17, 33), (37, 130), (100, 72), (300, 260)])
def test_ragged(M, N, split):
    note(f"ragged M={M} N={N} split={split}")
    xb, wb, perm = _rand_case(M, N, split, seed=M * 7 + N + split[0])
    _check_full(xb, wb, perm, split, f"M{M} N{N} {split}")


@pytest.mark.parametrize("formats", [("E3M2", "E4M3"), ("E2M3", "E5M2")], ids="-".join)
@pytest.mark.parametrize("M,N,split", FEW_STAGES, ids=str)
def test_tiled_few_stages(M, N, split, formats):
    """The LDS-tiled kernel's ring with fewer stages than slots, as many and a
    few more, groups of one stage and groups that change while the ring fills:
    256 x 128 tiles (loads by producer wavefronts) and, in the last two, 256 x 256
    tiles."""
    note(f"tiled M={M} N={N} split={split} {formats}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + N + split[0])
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split, formats=formats)
    w = b.quantize_weight(to_dev_bf16(wb), p, split, formats=formats)
    y = b.gemm(a, w)
    torch.cuda.synchronize()
    fm = (O.E2M1, O.FORMATS[formats[0]], O.FORMATS[formats[1]])
    ra, rw = O.quantize_mixed(xb, perm, split, fm), O.quantize_mixed(wb, perm, split, fm)
    assert_gemm_close(y_to_f64(y), O.gemm_mixed(ra, rw), ctx=f"{formats} M{M} N{N} {split}")


@pytest.mark.parametrize("M,N,split", [(1, 6001, (96, 160, 96)), (20, 6000, (256, 128, 128)),
                                       (50, 6000, (0, 0, 512)), (1, 12000, (256, 128, 128)),
                                       (20, 12000, (96, 160, 96)), (50, 12000, (256, 128, 128)),
                                       (8, 20008, (256, 128, 128)), (64, 20000, (0, 0, 512))])
def test_decode_strips(M, N, split):
    """At most 64 rows against weights of few channels: the decode kernel's 16-row
    strips (N = 6001) and whole 32-row groups (N = 12000, 20008: a part-filled last
    group) with one activation tile, and the K-splitting kernel's narrow tiles
    above 16 rows, with part-filled last tiles."""
    note(f"decode strips M={M} N={N} split={split}")
    xb, wb, perm = _rand_case(M, N, split, seed=M * 11 + N + split[0])
    _check_full(xb, wb, perm, split, f"M{M} N{N} {split}")


@pytest.mark.parametrize("M,N", [(4, 700), (24, 300)])
def test_decode_long_k(M, N):
    """Decode kernel on the MLP-down width (K = 14336, split 10752 / 2688 / 896:
    84, 21 and 7 steps): the eight wavefronts go 5 / 2 / 1 to the groups, so
    every group takes several batches of steps per wavefront."""
    split = (10752, 2688, 896)
    note(f"decode long K M={M} N={N}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + N)
    _check_full(xb, wb, perm, split, f"M{M} N{N} {split}")


@pytest.mark.parametrize("split", [(96, 160, 96), (352, 0, 0), (0, 352, 0), (0, 0, 352), (128, 0, 224)])
@pytest.mark.parametrize("M,N", [(3000, 5400), (1000, 1000)])
def test_ragged_large(M, N, split):
    """Every output of shapes of the LDS-tiled kernel (24 x 22 tiles of 256 x 128)
    and of the K-splitting one (16 x 16 tiles of 64 x 64), both with ragged last
    tiles in M and N."""
    note(f"ragged large M={M} N={N} split={split}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + N + split[1])
    _check_full(xb, wb, perm, split, f"M{M} N{N} {split}")


@pytest.mark.parametrize("M,N", [(3000, 5400), (1000, 1000)])
def test_ragged_large_alternative_formats(M, N):
    split, formats = (96, 160, 96), ("E2M3", "E5M2")
    note(f"ragged large formats {formats} M={M} N={N}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + 2 * N)
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split, formats=formats)
    w = b.quantize_weight(to_dev_bf16(wb), p, split, formats=formats)
    y = b.gemm(a, w)
    torch.cuda.synchronize()
    fm = (O.E2M1, O.FORMATS[formats[0]], O.FORMATS[formats[1]])
    ra, rw = O.quantize_mixed(xb, perm, split, fm), O.quantize_mixed(wb, perm, split, fm)
    assert_codes_equal(a, ra, ctx="A")
    assert_codes_equal(w, rw, ctx="W")
    assert_gemm_close(y_to_f64(y), O.gemm_mixed(ra, rw), ctx=f"{formats} M{M} N{N}")


@pytest.mark.parametrize("w", W.decode_workloads(), ids=lambda w: w.name)
def test_decode_configs(w):
    """Full activation and full weight on the GPU; oracle on 256 sampled
    weight rows (output columns), all activation rows."""
    note(w.name)
    xb, wb, perm = w.x_bits(), w.w_bits(), w.perm()
    a, wq = _gpu_pair(xb, wb, perm, w.split)
    y = _b().gemm(a, wq)
    torch.cuda.synchronize()
    cols = np.unique(np.concatenate([[0, w.N - 1], np.random.default_rng(2).choice(w.N, 254, replace=False)]))
    ra, rw = O.quantize_mixed(xb, perm, w.split), O.quantize_mixed(wb[cols], perm, w.split)
    assert_codes_equal(a, ra, ctx=w.name + " A")
    assert_codes_equal(wq, rw, rows=cols, ctx=w.name + " W")
    assert_gemm_close(y_to_f64(y)[:, cols], O.gemm_mixed(ra, rw), ctx=w.name)


@pytest.mark.parametrize("w", W.PREFILL, ids=lambda w: w.name)
def test_prefill_configs_sampled(w):
    """Full-size quantisers and GEMM on the GPU; the oracle quantises 64
    sampled activation rows and 64 sampled weight rows (their codes and
    scales must match the GPU's bytes) and recomputes the 64 x 64 outputs
    they meet in."""
    note(w.name)
    xb, wb, perm = w.x_bits(), w.w_bits(), w.perm()
    a, wq = _gpu_pair(xb, wb, perm, w.split)
    y = _b().gemm(a, wq)
    torch.cuda.synchronize()
    rng = np.random.default_rng(3)
    rows = np.unique(np.concatenate([[0, w.M - 1], rng.choice(w.M, 62, replace=False)]))
    cols = np.unique(np.concatenate([[0, w.N - 1], rng.choice(w.N, 62, replace=False)]))
    ra, rw = O.quantize_mixed(xb[rows], perm, w.split), O.quantize_mixed(wb[cols], perm, w.split)
    assert_codes_equal(a, ra, rows=rows, ctx=w.name + " A")
    assert_codes_equal(wq, rw, rows=cols, ctx=w.name + " W")
    assert_gemm_close(y_to_f64(y[torch.from_numpy(rows).cuda()])[:, cols], O.gemm_mixed(ra, rw), ctx=w.name)


@pytest.mark.parametrize("split", [(320, 256, 128), (704, 0, 0), (32, 672, 0), (0, 96, 608)], ids=str)
@pytest.mark.parametrize("M,N", [(17, 33), (32, 4100), (20, 9000), (33, 31), (65, 1003), (129, 2050), (192, 5500),
                                 (250, 4097)])
def test_split_k_tiles(M, N, split):
    """Sizes between the decode and the tiled kernel: above 64 rows the K-splitting
    kernel's tile shapes (32 or 64 weight rows by 32 to 96 activation rows), last
    tiles that reach back into the tile before in both directions,
    columns that are no multiple of 8, wavefronts without steps, with one and
    with an odd number of steps; below, the decode kernel's strips at the same
    sizes.  Every output against the oracle."""
    note(f"split-K M={M} N={N} split={split}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + 3 * N + split[0])
    _check_full(xb, wb, perm, split, f"M{M} N{N} {split}")


@pytest.mark.parametrize("formats", [("E3M2", "E4M3"), ("E2M3", "E5M2")], ids="-".join)
@pytest.mark.parametrize("M,N,split", [(500, 4090, (2304, 576, 192)), (97, 600, (9216, 3328, 1792)),
                                       (9, 9000, (5120, 1024, 512))], ids=str)
def test_split_k_long(M, N, split, formats):
    """The same with many steps per wavefront: the widest tile (64 x 128 at 500
    rows), odd step counts; and the decode kernel with 9 rows."""
    note(f"split-K long M={M} N={N} split={split} {formats}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + N)
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split, formats=formats)
    w = b.quantize_weight(to_dev_bf16(wb), p, split, formats=formats)
    y = b.gemm(a, w)
    torch.cuda.synchronize()
    fm = (O.E2M1, O.FORMATS[formats[0]], O.FORMATS[formats[1]])
    ra, rw = O.quantize_mixed(xb, perm, split, fm), O.quantize_mixed(wb, perm, split, fm)
    assert_gemm_close(y_to_f64(y), O.gemm_mixed(ra, rw), ctx=f"{formats} M{M} N{N}")


@pytest.mark.parametrize("M", [1, 16])
def test_split_k_decode(M):
    """At most 16 rows against a weight of 48 MB (256 sampled columns against the
    oracle)."""
    N, split = 20000, (3072, 768, 256)
    note(f"split-K decode M={M}")
    xb, wb, perm = _rand_case(M, N, split, seed=M)
    a, wq = _gpu_pair(xb, wb, perm, split)
    y = _b().gemm(a, wq)
    torch.cuda.synchronize()
    cols = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(2).choice(N, 254, replace=False)]))
    ra, rw = O.quantize_mixed(xb, perm, split), O.quantize_mixed(wb[cols], perm, split)
    assert_gemm_close(y_to_f64(y)[:, cols], O.gemm_mixed(ra, rw), ctx=f"M{M}")


def test_one_activation_feeds_two_weights():
    """One quantised activation reused by two GEMMs with the same sigma."""
    note("shared activation")
    split = (256, 64, 64)
    xb, wb, perm = _rand_case(40, 96, split, seed=5)
    _, wb2, _ = _rand_case(40, 48, split, seed=6)
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split)
    y1 = b.gemm(a, b.quantize_weight(to_dev_bf16(wb), p, split))
    y2 = b.gemm(a, b.quantize_weight(to_dev_bf16(wb2), p, split))
    torch.cuda.synchronize()
    ra = O.quantize_mixed(xb, perm, split)
    assert_gemm_close(y_to_f64(y1), O.gemm_mixed(ra, O.quantize_mixed(wb, perm, split)), "y1")
    assert_gemm_close(y_to_f64(y2), O.gemm_mixed(ra, O.quantize_mixed(wb2, perm, split)), "y2")


@pytest.mark.parametrize("formats", [("E2M3", "E5M2"), ("E2M3", "E4M3"), ("E3M2", "E5M2")], ids="-".join)
@pytest.mark.parametrize("M,N", [(5, 70), (37, 130), (300, 260)])
def test_alternative_formats(M, N, formats):
    """The ablation's MXFP6 = E2M3 and MXFP8 = E5M2 variants through the decode
    and the K-splitting kernel (every kernel: test_every_kernel)."""
    split = (96, 160, 96)
    note(f"formats {formats} M={M} N={N}")
    xb, wb, perm = _rand_case(M, N, split, seed=M * 11 + N)
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split, formats=formats)
    w = b.quantize_weight(to_dev_bf16(wb), p, split, formats=formats)
    y = b.gemm(a, w)
    torch.cuda.synchronize()
    fm = (O.E2M1, O.FORMATS[formats[0]], O.FORMATS[formats[1]])
    ra, rw = O.quantize_mixed(xb, perm, split, fm), O.quantize_mixed(wb, perm, split, fm)
    ctx = f"{formats} M{M} N{N}"
    assert_codes_equal(a, ra, ctx=ctx + " A")
    assert_codes_equal(w, rw, ctx=ctx + " W")
    assert_gemm_close(y_to_f64(y), O.gemm_mixed(ra, rw), ctx=ctx)


@pytest.mark.parametrize("formats", [("E3M2", "E4M3"), ("E2M3", "E4M3"), ("E3M2", "E5M2"), ("E2M3", "E5M2")], ids="-".join)
@pytest.mark.parametrize("name,M,N,split", CASES, ids=str)
def test_every_kernel(name, M, N, split, formats):
    """Every compiled kernel with every format set: the first and last 70 rows and
    columns and 60 others against the oracle."""
    note(f"{name} {formats} M={M} N={N} split={split}")
    xb, wb, perm = _rand_case(M, N, split, seed=M + N + split[2])
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split, formats=formats)
    w = b.quantize_weight(to_dev_bf16(wb), p, split, formats=formats)
    y = b.gemm(a, w)
    torch.cuda.synchronize()

    def some(n):
        return np.unique(np.clip(np.concatenate([np.arange(70), n - 1 - np.arange(70),
                                                 np.random.default_rng(n).choice(n, 60)]), 0, n - 1))

    rows, cols = some(M), some(N)
    fm = (O.E2M1, O.FORMATS[formats[0]], O.FORMATS[formats[1]])
    ra, rw = O.quantize_mixed(xb[rows], perm, split, fm), O.quantize_mixed(wb[cols], perm, split, fm)
    got = y_to_f64(y[torch.from_numpy(rows).cuda()])[:, cols]
    assert_gemm_close(got, O.gemm_mixed(ra, rw), ctx=f"{name} {formats}")


def test_mixed_formats_are_rejected():
    xb, wb, perm = _rand_case(8, 16, (96, 160, 96), seed=3)
    b = _b()
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, (96, 160, 96), formats=("E2M3", "E4M3"))
    w = b.quantize_weight(to_dev_bf16(wb), p, (96, 160, 96))
    with pytest.raises(b.MMError, match="MM_ERR_FORMAT"):
        b.gemm(a, w)


@pytest.mark.parametrize("M", [8, 300])
def test_stacked_qkv_equals_separate_gemms(M):
    """Q, K and V share the activation's sigma and split, so their weights can
    be stacked along N (Llama-3-8B: 4096 + 1024 + 1024 rows), quantised once and
    multiplied in one launch; each column slice of that product equals,
    bit for bit, the separate GEMM of the same quantised activation (every
    output element sums the same K blocks in the same order)."""
    b = _b()
    K, split, parts = 4096, (3072, 768, 256), (4096, 1024, 1024)
    rng = np.random.default_rng(M)
    xb = W.LLAMA_ATTN.x_bits(M)
    perm = W.LLAMA_ATTN.perm()
    ws = [W.f32_to_bf16_bits((rng.standard_normal((n, K)) * 0.02).astype(np.float32)) for n in parts]
    note(f"stacked QKV M={M}")
    p = to_dev_perm(perm)
    a = b.quantize_act(to_dev_bf16(xb), p, split)
    stacked = b.gemm(a, b.quantize_weight(to_dev_bf16(np.concatenate(ws)), p, split))
    sep = [b.gemm(a, b.quantize_weight(to_dev_bf16(wk), p, split)) for wk in ws]
    torch.cuda.synchronize()
    col = 0
    for n, y in zip(parts, sep):
        assert torch.equal(stacked[:, col:col + n], y), (M, col)
        col += n
    ref = O.gemm_mixed(O.quantize_mixed(xb, perm, split), O.quantize_mixed(ws[1], perm, split))
    assert_gemm_close(y_to_f64(sep[1]), ref, ctx="K slice")
