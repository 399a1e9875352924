"""The tile kernel of the matrix form (more than 16 columns), against the CPU oracle: every number of row and column tiles, runs of 128
columns that leave some of its four pairs of wavefronts without one, ragged runs, segments, activations at any alignment and any distance."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_06178_amd import binding as B
from paper_2310_06178_amd import inputs, torch_io
from test_gpu_parity import Y_OF_X, check, elem_bound, matrix_form, oracle_y, run_gpu

pytestmark = pytest.mark.gpu

CASES = [(m, k, b, xd, sg, {"panels_per_workgroup": r}, pad) for r in (1, 2, 3) for m, k, b, xd, sg, pad in [
    (1, 128, 17, "f16", 0, 0),                  # one run: a single pair works
    (64, 130, 32, "bf16", 0, 1),                # the ragged run of two columns goes first; activations at odd addresses
    (65, 2 * 128 + 126, 33, "f16", 0, 3), (193, 4 * 128, 64, "f16", 0, 8), (130, 5 * 128 + 8, 49, "bf16", 0, 0),
    (257, 12 * 128 + 66, 64, "i8", 0, 1), (200, 13 * 128, 50, "i8", 0, 2), (63, 9 * 128 + 14, 100, "i8", 0, 16), (129, 8 * 128 + 2, 65, "f16", 0, 7)]]
CASES += [(m, k, b, xd, sg, {"panels_per_workgroup": r}, 8) for r in (1, 2) for m, k, b, xd, sg in [
    (130, 3 * 128, 20, "f16", 128), (257, 14 * 128, 64, "bf16", 128), (100, 16 * 128, 33, "f16", 256), (64, 9 * 128, 90, "bf16", 384)]]
CASES += [(131, 11 * 128 + 2, b, xd, 0, {"batched_segments": s}, 3) for s in (2, 5, 12) for b, xd in ((24, "bf16"), (64, "f16"), (64, "i8"))]


@pytest.mark.parametrize("m,k,b,xd,sg,options,pad", CASES)
def test_against_oracle(m, k, b, xd, sg, options, pad):
    codes = inputs.make_codes(m, k, seed=m + 3 * k + b)
    X = inputs.make_x(k, b, xd, seed=k + b)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    out, info = run_gpu(codes, X, xd, scales, sg, 2, B.VARIANT_AUTO, ldx_pad=pad, ldy_pad=5, options=dict(options, batched_form=3, rows_per_lane=4))
    assert matrix_form(info)
    check(out, oracle_y(codes, X, xd, scales, sg), xd, f"{options}", elem_bound(codes, X, xd, scales, sg))


SHORT8 = [(11008, 1154, 20), (11008, 1024, 41), (33000, 130, 32)]


@pytest.mark.parametrize("m,k,b", SHORT8)
def test_int8_short_k_own_choice(m, k, b):
    """A short k under many rows goes to the tile kernel without being asked to, also with few columns (that it does: test_matrix_form_choice.py)."""
    codes, X = inputs.make_codes(m, k, seed=1), inputs.make_x(k, b, "i8", seed=2)
    out, info = run_gpu(codes, X, "i8", None, 0, 2, B.VARIANT_AUTO)
    assert matrix_form(info)
    check(out, oracle_y(codes, X, "i8", None, 0), "i8")


@pytest.mark.parametrize("xd", ["f16", "bf16"])
@pytest.mark.parametrize("b", [17, 40])
def test_nothing_behind_k_is_used(xd, b):
    """NaNs behind the last column of every row of X, k ending anywhere in a run."""
    m = 70
    for k in (130, 254, 386, 898, 1018):
        codes, X = inputs.make_codes(m, k, seed=k), inputs.make_x(k, b, xd, seed=5)
        Xp = np.zeros((b, k + 130), dtype=X.dtype)
        Xp.view(np.uint16)[:] = 0x7e01 if xd == "f16" else 0x7fc1
        Xp[:, :k] = X
        dX, Y = torch_io.to_device(Xp, xd), torch_io.empty_output(b, m, xd)
        plan = B.msgemm_plan(m, k, b, xd, xd, 2, 0, torch_io.to_device(codes, "codes"), options={"batched_form": 3, "rows_per_lane": 4})
        try:
            B.msgemm_run(plan, dX, k + 130, Y, m)
            torch.cuda.synchronize()
            check(torch_io.to_host(Y), oracle_y(codes, X, xd, None, 0), xd, f"k {k}", elem_bound(codes, X, xd, None, 0))
        finally:
            B.msgemm_destroy(plan)


@pytest.mark.parametrize("xd,b,sg,r", [("f16", 17, 0, 1), ("f16", 33, 128, 2), ("bf16", 33, 0, 3), ("bf16", 17, 128, 1), ("i8", 50, 0, 2)])
def test_rows_of_x_far_apart(xd, b, sg, r):
    """Rows of X gigabytes apart (more than the direct loads' 32-bit offsets reach), with a ragged run where there are no scales."""
    m, k = 200, 5 * 128 + (0 if sg else 34)
    size = 1 if xd == "i8" else 2
    ldx = 2 ** 31 // ((33 if b <= 32 else 65) * size) + 3
    codes, X = inputs.make_codes(m, k, seed=7), inputs.make_x(k, b, xd, seed=8)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    small = torch_io.to_device(X, xd)
    dX = torch.empty((b - 1) * ldx + k, dtype=small.dtype, device="cuda:0")
    for c in range(b):
        dX[c * ldx:c * ldx + k] = small[c]
    Y = torch_io.empty_output(b, m, Y_OF_X[xd])
    plan = B.msgemm_plan(m, k, b, xd, Y_OF_X[xd], 2, sg, torch_io.to_device(codes, "codes"), torch_io.to_device(scales, "scales"),
                         options={"batched_form": 3, "rows_per_lane": 4, "panels_per_workgroup": r})
    try:
        B.msgemm_run(plan, dX, ldx, Y, m)
        torch.cuda.synchronize()
        check(torch_io.to_host(Y), oracle_y(codes, X, xd, scales, sg), xd, "far apart", elem_bound(codes, X, xd, scales, sg))
    finally:
        B.msgemm_destroy(plan)


@pytest.mark.parametrize("xd,b,sg", [("f16", 20, 128), ("bf16", 64, 0), ("i8", 64, 0)])
def test_codes_come_back_from_its_order(xd, b, sg):
    """Entry points that read rows of codes make them from the tile kernel's order."""
    m, k, yd = 300, 1154 if not sg else 1152, Y_OF_X[xd]
    codes, X = inputs.make_codes(m, k, seed=1), inputs.make_x(k, b, xd, seed=2)
    scales = inputs.make_scales(m, k, sg, seed=3) if sg else None
    dX, Y = torch_io.to_device(X, xd), torch_io.empty_output(b, m, yd)
    plan = B.msgemm_plan(m, k, b, xd, yd, 2, sg, torch_io.to_device(codes, "codes"), torch_io.to_device(scales, "scales"),
                         options={"batched_form": 3, "rows_per_lane": 4})
    try:
        L = torch.empty(B.msgemm_lut_bytes(plan) // 4, dtype=torch.int32, device="cuda:0")
        B.msgemm_build_lut(plan, dX, k, L)
        B.msgemm_consume_lut(plan, L, Y, m)
        torch.cuda.synchronize()
        check(torch_io.to_host(Y), oracle_y(codes, X, xd, scales, sg), xd, "two phases", elem_bound(codes, X, xd, scales, sg))
    finally:
        B.msgemm_destroy(plan)


def test_replays_of_a_graph():
    m, k, b = 700, 1410, 64
    codes, X = inputs.make_codes(m, k, seed=1), inputs.make_x(k, b, "f16", seed=2)
    dX, Y = torch_io.to_device(X, "f16"), torch_io.empty_output(b, m, "f16")
    plan = B.msgemm_plan(m, k, b, "f16", "f16", 2, 0, torch_io.to_device(codes, "codes"), options={"batched_form": 3, "rows_per_lane": 4, "batched_segments": 3})
    try:
        B.msgemm_run(plan, dX, k, Y, m)
        torch.cuda.synchronize()
        first = torch_io.to_host(Y).copy()
        check(first, oracle_y(codes, X, "f16", None, 0), "f16", "eager", elem_bound(codes, X, "f16", None, 0))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            B.msgemm_run(plan, dX, k, Y, m)
        for _ in range(4):
            Y.fill_(-3)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(torch_io.to_host(Y), first)
    finally:
        B.msgemm_destroy(plan)


def _formats():
    from test_matrix_form import e5m2_values
    return {"e4m3": np.nan_to_num(inputs.fp8_e4m3_values(), nan=-0.5), "e5m2": e5m2_values()}


# (values up to 448: a result of 1666 of them times N(0, 1) has a deviation of 6000, a tenth of the largest fp16; times 2^3 it would be past it)
@pytest.mark.parametrize("table,power", [("e4m3", -4), ("e5m2", -12), ("e4m3", 0)])
@pytest.mark.parametrize("m,k,b,xd,sg,options,pad", [
    (m, k, b, xd, sg, {"panels_per_workgroup": r}, pad) for r in (1, 2) for m, k, b, xd, sg, pad in [
        (1, 128, 17, "f16", 0, 0), (130, 4 * 128 + 66, 32, "bf16", 0, 1), (200, 13 * 128 + 2, 64, "f16", 0, 7), (129, 9 * 128, 20, "bf16", 128, 8),
        (65, 10 * 128, 50, "f16", 256, 0), (70, 5 * 128, 90, "bf16", 128, 3)]] + [(131, 11 * 128 + 2, 33, "f16", 0, {"batched_segments": 5}, 0)])
def test_8_bit_codes_against_oracle(m, k, b, xd, sg, options, pad, table, power):
    values = _formats()[table] * 2.0 ** power
    codes = np.random.default_rng(m + k + b).integers(0, 256, size=(m, k), dtype=np.uint8)
    X = inputs.make_x(k, b, xd, seed=k + 1)
    Xp = np.zeros((b, k + pad), dtype=X.dtype)
    Xp[:, :k], Xp[:, k:] = X, 77 if xd == "f16" else 0x4300
    scales = inputs.make_scales(m, k, sg, seed=10) if sg else None
    Xd = oracle.bf16_bits_to_f64(X) if xd == "bf16" else X.astype(np.float64)
    ref = oracle.gemm_f64_codes8(codes, Xd, values, scales, sg)
    plan = B.msgemm_plan_codes8(m, k, b, xd, Y_OF_X[xd], sg, torch_io.to_device(codes, "codes"), torch_io.to_device(scales, "scales"), values,
                                options=dict(options, batched_form=3, rows_per_lane=4))
    try:
        Y = torch_io.empty_output(b, m, Y_OF_X[xd], ldy=m + 1)
        Y.fill_(-3)
        B.msgemm_run(plan, torch_io.to_device(Xp, xd), k + pad, Y, m + 1)
        torch.cuda.synchronize()
        out = torch_io.to_host(Y)
    finally:
        B.msgemm_destroy(plan)
    check(np.ascontiguousarray(out[:, :m]), ref, xd, f"8-bit weights {table}", elem_bound(codes, X, xd, scales, sg, values256=values))


# (1e-36 times the map's own values: results that stay normal numbers)
@pytest.mark.parametrize("xd,magnitude,power", [("bf16", 1e35, -20), ("bf16", 1e35, -12), ("bf16", 1e-36, 0), ("f16", 1e2, -20), ("f16", 1e2, -12)])
@pytest.mark.parametrize("b,sg", [(20, 0), (40, 128)])
def test_8_bit_codes_at_the_ends_of_the_range(b, sg, power, xd, magnitude):
    m, k = 64, 1280 if sg else 1282
    values = _formats()["e5m2"] * 2.0 ** power
    codes = np.random.default_rng(m + b).integers(0, 256, size=(m, k), dtype=np.uint8)
    X = (inputs.make_x(k, b, "f32", seed=k + 1) * np.float32(magnitude)).astype(np.float32)
    X = inputs.f32_to_bf16_bits(X) if xd == "bf16" else X.astype(np.float16)
    scales = inputs.make_scales(m, k, sg, seed=10) if sg else None
    Xd = oracle.bf16_bits_to_f64(X) if xd == "bf16" else X.astype(np.float64)
    ref = oracle.gemm_f64_codes8(codes, Xd, values, scales, sg)
    assert np.abs(ref).max() < {"f16": 6.5e4, "bf16": 3e38}[xd]
    plan = B.msgemm_plan_codes8(m, k, b, xd, Y_OF_X[xd], sg, torch_io.to_device(codes, "codes"), torch_io.to_device(scales, "scales"), values,
                                options={"batched_form": 3, "rows_per_lane": 4})
    try:
        Y = torch_io.empty_output(b, m, Y_OF_X[xd])
        B.msgemm_run(plan, torch_io.to_device(X, xd), k, Y, m)
        torch.cuda.synchronize()
        out = torch_io.to_host(Y)
    finally:
        B.msgemm_destroy(plan)
    check(out, ref, xd, f"E5M2 times 2^{power}", elem_bound(codes, X, xd, scales, sg, values256=values))
