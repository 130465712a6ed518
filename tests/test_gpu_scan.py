"""S1 parity: the HIP top-M + tail-LSE scan against the oracle (Alg. 1 step 1; section 3.2).

Token ids and their logits must match exactly (pure comparisons of exact
values, ties by lower id); the tail log-sum-exp within 1e-5 relative.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_util import to_dev
from paper_2607_08642_amd import binding, synth

pytestmark = pytest.mark.gpu


def _check(x_np, dtype, M, T, rows=None, case=""):
    print(f"[scan] {case} shape={x_np.shape} dtype={dtype} M={M} T={T}", flush=True)
    x = to_dev(x_np, dtype)
    ids, vals, tail, flags = binding.scan_topm(x, M, T)
    torch.cuda.synchronize()
    ids, vals, tail, flags = (a.cpu().numpy() for a in (ids, vals, tail, flags))
    Xw = oracle.widen(x_np, dtype)
    tau = oracle.effective_temperature(T)
    for r in (range(x_np.shape[0]) if rows is None else rows):
        bad = bool(np.any(np.isnan(Xw[r])) or np.any(Xw[r] == np.inf))
        assert flags[r] == (oracle.TREE_NONFINITE if bad else 0), (case, r)
        if bad:
            continue
        rid, rx, rR = oracle.scan_row(Xw[r], M, tau)
        np.testing.assert_array_equal(ids[r], rid, err_msg=f"{case} row {r} ids")
        np.testing.assert_array_equal(vals[r].astype(np.float64), rx, err_msg=f"{case} row {r} vals")
        if rR == -math.inf:
            assert tail[r] == -np.inf
        else:
            assert abs(tail[r] - rR) <= 1e-5 * max(1.0, abs(rR)), (case, r, tail[r], rR)


def test_scan_tiny_fp32():
    wl = synth.tiny()
    _check(wl.logits[0], synth.DT_F32, 8, 0.0, case="tiny")


@pytest.mark.parametrize("T", [0.0, 1.0, 0.7, 0.05, 4.0])
def test_scan_qwen_rows_bf16(T):
    x = synth.peaked_logits(2, 0, 16, synth.QWEN3_VOCAB, synth.DT_BF16, 1, 4, 6.0, 12.0)
    _check(x, synth.DT_BF16, 64, T, case="qwen16")


@pytest.mark.parametrize("T", [0.05, 4.0])
def test_scan_block_kernel_temperatures(T):
    # rows of an odd length (most begin off a 16-byte boundary), M above and below
    # 64, at a small temperature (exponents far below the row maximum) and a
    # large one
    x = synth.peaked_logits(3, 0, 8, 20001, synth.DT_F32, 1, 4, 6.0, 12.0)
    _check(x, synth.DT_F32, 100, T, case=f"block M=100 T={T}")
    _check(x, synth.DT_F32, 32, T, case=f"block M=32 T={T}")


def test_scan_concurrent_rows_sampled():
    x = np.concatenate([synth.peaked_logits(4, t, 16, synth.QWEN3_VOCAB, synth.DT_BF16, 1, 4,
                                            6.0, 12.0) for t in range(32)])
    _check(x, synth.DT_BF16, 64, 0.7, rows=list(range(0, 512, 17)) + [511], case="concurrent")


def test_scan_flattened_rows_bf16():
    x = synth.peaked_logits(3, 0, 16, synth.QWEN3_VOCAB, synth.DT_BF16, 4, 16, 3.0, 6.0)
    _check(x, synth.DT_BF16, 64, 0.0, case="flattened")


def test_scan_heavy_ties():
    rng = np.random.default_rng(5)
    x = np.round(rng.standard_normal((6, 20000)) * 3).astype(np.float32)   # integers: huge ties
    _check(x, synth.DT_F32, 64, 1.0, case="ties-f32")
    _check(synth.f32_to_bf16_bits(x), synth.DT_BF16, 200, 0.5, case="ties-bf16")


def test_scan_all_equal_and_neg_inf():
    x = np.zeros((3, 5000), np.float32)
    x[1, ::3] = -np.inf
    x[2, :] = -np.inf
    x[2, 4000:4003] = 1.0
    _check(x, synth.DT_F32, 16, 0.0, case="equal/-inf")


@pytest.mark.parametrize("V,M", [(1001, 7), (3, 3), (64, 64), (257, 256), (9000, 1)])
def test_scan_odd_shapes(V, M):
    rng = np.random.default_rng(V)
    x = (rng.standard_normal((5, V)) * 2).astype(np.float32)
    _check(x, synth.DT_F32, M, 0.0, case=f"f32 V={V}")
    _check(synth.f32_to_bf16_bits(x), synth.DT_BF16, M, 0.9, case=f"bf16 V={V}")


def test_scan_descending_rows_worst_case():
    # increasing values: every sub-batch beats the running threshold
    V = 40000
    x = np.tile(np.arange(V, dtype=np.float32) / 100.0, (2, 1))
    x[1] = x[1][::-1]
    _check(x, synth.DT_F32, 256, 1.0, case="monotone")


def test_scan_nonfinite_flags():
    rng = np.random.default_rng(9)
    x = rng.standard_normal((5, 3000)).astype(np.float32)
    x[1, 17] = np.nan
    x[2, 2999] = np.inf
    # a first batch without a finite lower bound, holding a NaN
    x[3, :] = -np.inf
    x[3, 5] = np.nan
    x[3, 2500] = 1.0
    _check(x, synth.DT_F32, 8, 0.0, case="nonfinite")


def _mixed_rows(n_rows, V, seed):
    """Rows of several kinds: normal, integer ties, rising and falling ramps,
    constant, -inf blocks, a late spike."""
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((n_rows, V)) * 2).astype(np.float32)
    kinds = np.arange(n_rows) % 7
    ramp = np.arange(V, dtype=np.float32) / 64.0
    x[kinds == 1] = np.round(x[kinds == 1] * 2)
    x[kinds == 2] = ramp
    x[kinds == 3] = ramp[::-1]
    x[kinds == 4] = 0.5
    blk = np.flatnonzero(kinds == 5)
    x[blk, : V // 3] = -np.inf
    late = np.flatnonzero(kinds == 6)
    x[late, V - 5] = 40.0
    return x


@pytest.mark.parametrize("V", [20480 + 37, 20480 + 40], ids=["unaligned", "aligned"])
@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
def test_scan_streaming_segments(dtype, V):
    # enough rows that every workgroup streams several batches of a segment
    # against its running lists (ramps and constant rows overflow the candidate
    # regions; -inf blocks leave first batches without a finite bound), with one
    # list register per lane (M <= 64) and with four.
    x = _mixed_rows(1100, V, 21)
    if dtype == synth.DT_BF16:
        x = synth.f32_to_bf16_bits(x)
    rows = list(range(0, 14)) + list(range(500, 507)) + [1099]
    _check(x, dtype, 64, 0.8, rows=rows, case=f"streaming {dtype}")
    _check(x, dtype, 200, 0.0, rows=rows[:7], case=f"streaming M=200 {dtype}")


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
def test_scan_neg_inf_prefixes(dtype):
    # Segments of four batches (1100 rows of 30760) whose first batch, or first
    # two batches, hold no finite value: the first bound then comes from the
    # second batch alone, or from neither (every element of the first batch is
    # taken as a candidate and the finite ones arrive through overflowing
    # regions later); and rows with fewer finite values than M.
    V = 30720 + 40
    x = (np.random.default_rng(5).standard_normal((1100, V)) * 2).astype(np.float32)
    kinds = np.arange(1100) % 5
    x[kinds == 1, :10240] = -np.inf
    x[kinds == 2, : 20480 + 100] = -np.inf
    x[kinds == 3, : V - 20] = -np.inf
    x[kinds == 4, 10240:20480] = -np.inf
    if dtype == synth.DT_BF16:
        x = synth.f32_to_bf16_bits(x)
    rows = list(range(0, 10)) + [1095, 1096, 1097, 1098, 1099]
    _check(x, dtype, 64, 0.8, rows=rows, case=f"-inf prefixes {dtype}")
    _check(x, dtype, 32, 0.0, rows=rows[:5], case=f"-inf prefixes M=32 {dtype}")


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
def test_scan_large_magnitudes(dtype):
    # logits far from zero (an offset of 5000, a spread of hundreds): the
    # exponent's fma form does not apply (|m c| > 128), and the bf16 rows (a
    # spacing of 32 at 5000) are full of exact ties
    x = synth.peaked_logits(4, 0, 8, 30720 + 40, synth.DT_F32, 1, 4, 6.0, 12.0) * 150.0 + 5000.0
    x = x.astype(np.float32)
    if dtype == synth.DT_BF16:
        x = synth.f32_to_bf16_bits(x)
    _check(x, dtype, 64, 1.0, case=f"large {dtype}")
    _check(x, dtype, 64, 40.0, case=f"large T=40 {dtype}")


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
def test_scan_waves_without_enough_finite_lanes(dtype):
    # finite values only in the elements one wave of the first batch reads
    # (the first 300 of each 2048), so the other waves' bound inputs are -inf:
    # the segment's bound must then be -inf (every element a candidate), not
    # that wave's; one- and two-batch segments, rows on and off a 16-byte boundary
    rng = np.random.default_rng(9)
    for V in (10240, 20480, 10243):
        x = np.full((6, V), -np.inf, np.float32)
        for j in range(0, V, 2048):
            x[:, j : j + 300] = (rng.standard_normal((6, min(300, V - j))) * 2).astype(np.float32)
        xd = synth.f32_to_bf16_bits(x) if dtype == synth.DT_BF16 else x
        _check(xd, dtype, 64, 0.9, case=f"sparse waves V={V} {dtype}")


@pytest.mark.parametrize("dtype", [synth.DT_F32, synth.DT_BF16])
def test_scan_signed_zeros(dtype):
    # -0 and +0 are one value: ties between them go to the lower id
    x = np.zeros((3, 20480 + 64), np.float32)
    x[:, ::2] = -0.0
    x[0, 7] = 1.0
    x[1, 100:140] = -1.0
    x[2, ::3] = -np.inf
    xd = synth.f32_to_bf16_bits(x) if dtype == synth.DT_BF16 else x
    _check(xd, dtype, 64, 1.0, case=f"signed zeros {dtype}")
    _check(xd, dtype, 200, 0.5, case=f"signed zeros M=200 {dtype}")


@pytest.mark.parametrize("dtype,per", [(synth.DT_BF16, 8), (synth.DT_F32, 4)], ids=["bf16", "fp32"])
@pytest.mark.parametrize("M", [1, 64, 65, 128, 129, 256])
def test_scan_rows_at_any_offset(dtype, per, M):
    # rows that begin at every element of a 16-byte granule, of lengths just around
    # whole batches and granules and below one granule, between NaNs that no row may
    # read: the same ids and values as the oracle, and the tail within its rounding
    base = synth.peaked_logits(11, 0, 4, 3 * 10240 + 16, dtype, 1, 4, 6.0, 12.0)
    for off, V in [(0, 10240), (1, 10239), (per - 1, 10241), (3, 20480 + per - 1), (2, 257),
                   (1, max(M, per - 1)), (per // 2, 30720 + 1)]:
        if V < M:
            continue
        rows = np.ascontiguousarray(base[:3, :V])
        x = to_dev(rows, dtype)
        buf = torch.full((x.numel() + 2 * per,), float("nan"), dtype=x.dtype, device=x.device)
        view = buf[off:off + x.numel()].view(3, V)
        view.copy_(x)
        print(f"[scan] offset {off} V={V} M={M} dtype={dtype}", flush=True)
        ids, vals, tail, flags = (a.cpu().numpy() for a in binding.scan_topm(view, M, 0.7))
        X = oracle.widen(rows, dtype)
        assert not flags.any(), (off, V)
        for r in range(3):
            rid, rx, rR = oracle.scan_row(X[r], M, oracle.effective_temperature(0.7))
            np.testing.assert_array_equal(ids[r], rid, err_msg=f"offset {off} V {V} row {r}")
            np.testing.assert_array_equal(vals[r].astype(np.float64), rx)
            # fp32 sums of V terms over 256 threads and a tree: (V / 256 + 16) roundings of 2^-24,
            # each term exact to a few ulps of its exponent
            assert tail[r] == rR or abs(tail[r] - rR) <= (V / 256 + 64) * 2.0 ** -24 * max(1.0, abs(rR)), (off, V, r)


@pytest.mark.parametrize("M", [1, 63, 64, 65, 128, 129, 256])
@pytest.mark.parametrize("nlists", [2, 3, 4, 5, 9, 21])
def test_scan_merge_of_many_segments(nlists, M):
    # two rows are cut into one segment per 10240 elements: fewer lists than waves,
    # as many, and several per wave, the last list shorter than M; runs of ties cross
    # the segments, one row's best values all lie in one segment
    V = (nlists - 1) * 10240 + max(1, M // 2)
    x = synth.peaked_logits(12, 0, 2, V, synth.DT_F32, 1, 4, 6.0, 12.0).reshape(2, V)
    x[0, ::641] = 14.0
    x[1, 10200:10200 + min(300, V - 10200)] += 30.0
    _check(x, synth.DT_F32, M, 1.0, case=f"{nlists} lists M={M}")


@pytest.mark.parametrize("dtype", [synth.DT_BF16, synth.DT_F32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("M", [1, 4, 64, 65, 256])
def test_scan_many_infinities(M, dtype):
    # rows of nothing but +inf, and rows that hold it often enough to make the first
    # batches' bound +inf itself: flagged, in one segment and several, beside rows
    # that are not
    for V in (257, 4099, 10240, 20481, 5 * 10240 + 3):
        x = synth.peaked_logits(13, 0, 6, V, synth.DT_F32, 1, 4, 6.0, 12.0).reshape(6, V)
        x[1, :] = np.inf
        x[2, ::3] = np.inf
        x[3, :] = -np.inf
        x[3, ::2] = np.inf
        x[4, V // 2:] = np.inf
        xd = synth.f32_to_bf16_bits(x) if dtype == synth.DT_BF16 else x
        _check(xd, dtype, M, 0.7, case=f"infinities V={V} M={M}")
