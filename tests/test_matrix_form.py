"""The matrix form of msgemm_run (codes decoded in registers, sums on the matrix cores), against the CPU oracle at the
sizes where its kernels can go wrong: edges of the 16-row tiles and of the 128-column runs, ragged last runs of a few
columns, every operand width (compact, 8, 16 and up to 64 columns, column passes), k cut into segments, unaligned activations,
infinities, NaNs, activations near the ends of their range."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2310_06178_amd import binding as B
from paper_2310_06178_amd import inputs, torch_io
from test_gpu_parity import ABS_FLOOR, NONUNIFORM, TOL, U_OUT, Y_OF_X, check, elem_bound, matrix_form, oracle_y, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    # m, k, b, xd, sg, options
    (1, 2, 1, "f32", 0, {}),
    (17, 126, 3, "f16", 0, {}),                 # no full run at all
    (15, 128, 4, "bf16", 128, {}),
    (65, 130, 2, "i8", 0, {}),
    (33, 258, 5, "f16", 0, {}),                 # a ragged run of two columns
    (64, 1152, 8, "bf16", 128, {}),             # nine runs over four wavefronts
    (129, 642, 9, "i8", 0, {}),
    (200, 1410, 16, "f32", 0, {}),
    (47, 384, 12, "f32", 384, {}),              # one scale per row
    (100, 2304, 1, "f32", 256, {}),
    (77, 5000, 7, "f32", 0, {}),
    (513, 4096, 16, "bf16", 256, {}),
    (300, 4098, 11, "f16", 0, {}),
] + [(m, k, b, xd, sg, {"panels_per_workgroup": r}) for r in (1, 2, 4) for m, k, b, xd, sg in [
    (131, 1666, 1, "f16", 0), (131, 1666, 8, "i8", 0), (131, 1666, 16, "i8", 0), (260, 1280, 6, "bf16", 128),
    (260, 1280, 4, "f32", 128), (100, 900, 14, "f16", 0)]
] + [(m, k, b, xd, sg, {"batched_segments": s}) for s in (2, 7) for m, k, b, xd, sg in [
    (131, 1154, 3, "f16", 0), (131, 1154, 16, "i8", 0), (70, 2560, 9, "bf16", 128), (70, 2050, 2, "f32", 0)]]


# more than 16 columns: the tile kernel (rows_per_lane 4) and passes of the streaming kernel (8)
CASES += [(m, k, b, xd, sg, {"rows_per_lane": 4, "panels_per_workgroup": r}) for r in (1, 2, 3) for m, k, b, xd, sg in [
    (1, 128, 17, "f16", 0),                     # one full run: padded steps only
    (63, 130, 32, "bf16", 0),                   # a ragged run of two columns after it
    (193, 1666, 33, "f16", 0), (193, 1666, 47, "i8", 0), (257, 898, 64, "i8", 0), (130, 1536, 20, "bf16", 128),
    (385, 1664, 65, "f16", 128),                # two column passes, the second of one column; 13 runs: 6.5 steps a group
    (65, 1792, 48, "bf16", 256)]
] + [(m, k, b, xd, sg, {"rows_per_lane": 4, "batched_segments": s}) for s in (2, 5) for m, k, b, xd, sg in [
    (131, 1154, 33, "f16", 0), (131, 1154, 64, "i8", 0), (70, 2560, 90, "bf16", 128)]
] + [(m, k, b, xd, sg, {"rows_per_lane": 8}) for m, k, b, xd, sg in [
    (131, 1154, 17, "f16", 0), (65, 1154, 35, "i8", 0), (70, 2560, 32, "bf16", 128), (100, 770, 50, "f32", 0)]
] + [(131, 1154, 33, "f16", 0, {"rows_per_lane": 8, "batched_segments": 3})]


@pytest.mark.parametrize("m,k,b,xd,sg,options", CASES)
def test_matrix_form_against_oracle(m, k, b, xd, sg, options):
    codes = inputs.make_codes(m, k, seed=m + 3 * k + b)
    X = inputs.make_x(k, b, xd, seed=k + b)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    out, info = run_gpu(codes, X, xd, scales, sg, 2, B.VARIANT_AUTO, ldx_pad=3, ldy_pad=5,
                        options=dict(options, batched_form=3))
    assert info["variant"] == B.VARIANT_FUSED_LDS and info["tile_groups"] == 64
    # full-width arithmetic: exact weights and products, fp32 sums
    check(out, oracle_y(codes, X, xd, scales, sg), xd, f"matrix form {options}", elem_bound(codes, X, xd, scales, sg))


def test_matrix_form_int8_sums_outgrow_the_shifted_accumulators():
    """The int8 kernel adds 16 x the products: over 2^31 / (16 * 1024) columns of the largest products it must have
    shifted back in between.  One segment of k = 300000 under one row tile, every sum at its largest."""
    m, k, b = 5, 300000, 2
    codes = np.full((m, k // 2), 0x88, dtype=np.uint8)
    X = np.full((b, k), -128, dtype=np.int8)
    X[1] = 127
    out, _ = run_gpu(codes, X, "i8", None, 0, 2, B.VARIANT_AUTO, options={"batched_form": 3, "batched_segments": 1})
    assert np.all(out[0] == 1024 * k) and np.all(out[1] == -8 * 127 * k)


@pytest.mark.parametrize("xd", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("b", [1, 6, 13, 20])
def test_matrix_form_infinite_activations(xd, b):
    """0 x inf is NaN and every other code gives an infinity of its sign, in the column that holds the infinity only."""
    m, k = 64, 512
    codes = inputs.make_codes(m, k, seed=4)
    X = inputs.make_x(k, b, "f32", seed=5)
    X[b - 1, 77] = np.inf
    Xh = {"f32": X, "f16": X.astype(np.float16), "bf16": inputs.f32_to_bf16_bits(X)}[xd]
    out, _ = run_gpu(codes, Xh, xd, None, 0, 2, B.VARIANT_AUTO, options={"batched_form": 3, "rows_per_lane": 4})
    y = torch_io.to_f64(out)
    v = np.array([oracle.decode(int(c)) for c in codes[:, 77 // 2] >> 4], dtype=np.float64)
    assert np.all(np.isnan(y[b - 1][v == 0])) and np.all(y[b - 1][v != 0] == np.inf * v[v != 0])
    assert np.all(np.isfinite(y[: b - 1]))


WIDTHS_F32 = [(b, sg, dict(o, batched_form=3)) for sg in (0, 128) for b, o in [
    (1, {}), (6, {}), (13, {}), (13, {"batched_segments": 2}), (2, {"batched_segments": 3}), (20, {}),
    (4, {"panels_per_workgroup": 2}), (4, {"panels_per_workgroup": 4}), (16, {"panels_per_workgroup": 2}),
    (16, {"panels_per_workgroup": 4})]]


@pytest.mark.parametrize("xd,magnitude", [("f32", 1e-30), ("f32", 1e-34), ("f32", 1e-36), ("f32", 3e-38), ("f32", 1e-40),
                                          ("f32", 1e37), ("bf16", 1e-37), ("bf16", 1e37)])
@pytest.mark.parametrize("b,sg,options", WIDTHS_F32)
def test_matrix_form_activations_of_any_magnitude(b, sg, options, xd, magnitude):
    """Activations near the ends of the range, subnormal ones among them: the bounds are those of ordinary ones (fp32: the
    products of the three parts are exact wherever the element is)."""
    m, k = 70, 1280 if sg else 1282
    codes = inputs.make_codes(m, k, seed=4)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    X = (inputs.make_x(k, b, "f32", seed=5) * np.float32(magnitude if magnitude < 1 else magnitude / 64)).astype(np.float32)
    if xd == "bf16":
        X = inputs.f32_to_bf16_bits(X)
    out, _ = run_gpu(codes, X, xd, scales, sg, 2, B.VARIANT_AUTO, options=options, ldx_pad=3)
    ref, bound = oracle_y(codes, X, xd, scales, sg), elem_bound(codes, X, xd, scales, sg)
    if magnitude < 1e-30:
        # results that are subnormal themselves: every rounding of a sum may be half a step of the format, with k / 32 + 8
        # of them per output (one per run and wavefront, and those inside an instruction)
        bound = bound + (k // 32 + 8) * 2.0 ** -150
        y = torch_io.to_f64(out)
        assert np.all(np.abs(y - ref) <= bound + U_OUT[xd] * 1.01 * np.abs(ref) + ABS_FLOOR[xd])
        if magnitude > 1e-39 and not sg:
            assert oracle.rel_l2(y, ref) <= TOL[xd]
    else:
        check(out, ref, xd, f"magnitude {magnitude}", bound)


@pytest.mark.parametrize("b,sg,options", [w for w in WIDTHS_F32 if w[0] > 1])
def test_matrix_form_infinity_beside_very_small_activations(b, sg, options):
    m, k = 70, 1280 if sg else 1282
    codes = inputs.make_codes(m, k, seed=4)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    X = (inputs.make_x(k, b, "f32", seed=5) * np.float32(1e-35)).astype(np.float32)
    ref, bound = oracle_y(codes, X, "f32", scales, sg), elem_bound(codes, X, "f32", scales, sg)
    X[b - 1, 500] = np.inf
    out, _ = run_gpu(codes, X, "f32", scales, sg, 2, B.VARIANT_AUTO, options=options)
    check(np.ascontiguousarray(out[:-1]), ref[:-1], "f32", "other columns", bound[:-1])
    v = np.array([oracle.decode(int(c)) for c in codes[:, 250] & 15], dtype=np.float64)
    assert np.array_equal(np.isnan(out[-1]), v == 0) and np.all(out[-1][v != 0] == np.inf * v[v != 0])


@pytest.mark.parametrize("b,sg,options", WIDTHS_F32)
def test_matrix_form_fp32_single_activations_are_exact(b, sg, options):
    """One activation at a time among zeros, from the smallest subnormal to the largest numbers, with patterns that fill
    all three parts: a product with a code is exact where fp32 can hold it, else within the step that two roundings can
    make.  A large one among codes of zero and other magnitudes in the other columns of X do not change that."""
    m, k = 16, 256
    codes = np.zeros((m, k // 2), dtype=np.uint8)
    codes[:, 36] = np.arange(16) | np.arange(16) << 4        # columns 72 and 73
    scales = np.full((m, k // sg), 0.5, dtype=np.float16) if sg else None
    patterns = [1 << i for i in (0, 1, 7, 8, 15, 16, 22)] + [0x00000fff, 0x000abcde, 0x007fffff, 0x00891a29, 0x00ffffff, 0x01fedcbb,
                                                            0x08abcdef, 0x0bffffff, 0x1f765432, 0x3f800001, 0x7cabcdef]
    value = np.array([oracle.decode(i) for i in range(16)], dtype=np.float64)
    for n in range(0, len(patterns), 1 if b == 1 else b):
        X = np.zeros((b, k), dtype=np.uint32)
        mine = (patterns + patterns)[n:n + b]
        X[:, 72], X[:, 200] = mine, 0x7cffffff               # (the second meets codes of zero)
        X = X.view(np.float32)
        out, _ = run_gpu(codes, X, "f32", scales, sg, 2, B.VARIANT_AUTO, options=options)
        ref = X[:, 72].astype(np.float64)[:, None] * value[None, :] * (0.5 if sg else 1.0)
        held = ref.astype(np.float32).astype(np.float64) == ref
        step = np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
        assert np.all(np.abs(out - ref) <= np.where(held, 0.0, step)), [hex(p) for p in mine]


# an operand width of each kind (compact, 8, 16 columns, the tile kernel, passes of the streaming kernel), with and
# without scales, in one segment and in several
SPECIAL = [(b, sg, dict(o, batched_form=3)) for sg in (0, 128) for b, o in [
    (1, {}), (6, {}), (13, {}), (13, {"batched_segments": 2}), (2, {"batched_segments": 3}), (20, {"rows_per_lane": 4}),
    (37, {"rows_per_lane": 4, "batched_segments": 2}), (20, {"rows_per_lane": 8})]]


@pytest.mark.parametrize("xd,bits", [("f32", 0x7f800001), ("f32", 0xff80ffff), ("f32", 0x7fc00000), ("f32", 0x7f810000),
                                     ("f16", 0x7c01), ("f16", 0xfe00), ("bf16", 0xff81), ("bf16", 0x7fc0)])
@pytest.mark.parametrize("b,sg,options", SPECIAL)
def test_matrix_form_nan_activations(b, sg, options, xd, bits):
    """A NaN, quiet or signalling, its payload in any bit, makes every output of its column a NaN (0 x NaN too), in a full
    run of columns and in a ragged one, and no other column's."""
    m, k = 70, 640 if sg else 642
    codes = inputs.make_codes(m, k, seed=4)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    for c, j in ((b - 1, k - 1), (0, 300)):
        X = inputs.make_x(k, b, xd, seed=5)
        X.view(np.uint32 if xd == "f32" else np.uint16)[c, j] = bits
        out, _ = run_gpu(codes, X, xd, scales, sg, 2, B.VARIANT_AUTO, options=options)
        y = torch_io.to_f64(out)
        assert np.all(np.isnan(y[c])) and np.all(np.isfinite(np.delete(y, c, axis=0)))


@pytest.mark.parametrize("xd", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("b,sg,options", [s for s in SPECIAL if s[1] or "batched_segments" in s[2]])
def test_matrix_form_infinite_activations_scaled_or_in_segments(b, sg, options, xd):
    m, k = 70, 640 if sg else 642
    codes = inputs.make_codes(m, k, seed=4)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None   # (positive)
    X = inputs.make_x(k, b, "f32", seed=5)
    X[b - 1, k - 2], X[0, 77] = -np.inf, np.inf
    Xh = {"f32": X, "f16": X.astype(np.float16), "bf16": inputs.f32_to_bf16_bits(X)}[xd]
    out, _ = run_gpu(codes, Xh, xd, scales, sg, 2, B.VARIANT_AUTO, options=options)
    y = torch_io.to_f64(out)
    terms = np.zeros((b, m))
    for c, j in ((0, 77), (b - 1, k - 2)):
        v = np.array([oracle.decode(int(c)) for c in codes[:, j // 2] >> (4 * (j & 1)) & 15], dtype=np.float64)
        with np.errstate(invalid="ignore"):
            terms[c] += X[c, j].astype(np.float64) * v
    assert np.array_equal(np.isnan(y), np.isnan(terms))
    hit = np.isinf(terms)
    assert np.array_equal(y[hit], terms[hit]) and np.all(np.isfinite(y[terms == 0]))


@pytest.mark.parametrize("xd,b,sg", [("f16", 1, 128), ("bf16", 5, 0), ("f32", 2, 0), ("i8", 16, 0)])
def test_other_entry_points_on_a_matrix_form_plan(xd, b, sg):
    """The library's own choice for this problem is the matrix form: phase 2 alone, the entry point that allocates
    nothing and another value map (served by the table kernels until the paper's map is restored) work on its plan."""
    m, k, yd = 300, 1154 if not sg else 1152, Y_OF_X[xd]
    codes = inputs.make_codes(m, k, seed=1)
    X = inputs.make_x(k, b, xd, seed=2)
    scales = inputs.make_scales(m, k, sg, seed=3) if sg else None
    ref, bound = oracle_y(codes, X, xd, scales, sg), elem_bound(codes, X, xd, scales, sg)
    dX = torch_io.to_device(X, xd)
    plan = B.msgemm_plan(m, k, b, xd, yd, 2, sg, torch_io.to_device(codes, "codes"), torch_io.to_device(scales, "scales"))
    try:
        def run(call):
            Y = torch_io.empty_output(b, m, yd)
            Y.fill_(-3)
            call(Y)
            torch.cuda.synchronize()
            return torch_io.to_host(Y)

        assert B.msgemm_plan_get_info(plan)["tile_groups"] == 64
        first = run(lambda Y: B.msgemm_run(plan, dX, k, Y, m))
        check(first, ref, xd, "matrix form", bound)
        assert np.array_equal(run(lambda Y: B.msgemm_run_static(plan, dX, k, Y, m)), first)
        L = torch.empty(B.msgemm_lut_bytes(plan) // 4, dtype=torch.int32, device="cuda:0")
        B.msgemm_build_lut(plan, dX, k, L)
        check(run(lambda Y: B.msgemm_consume_lut(plan, L, Y, m)), ref, xd, "two phases", bound)
        if xd != "i8":
            B.msgemm_plan_set_codebook(plan, NONUNIFORM)
            want = oracle.gemm_f64(codes, oracle.bf16_bits_to_f64(X) if xd == "bf16" else X.astype(np.float64), scales, sg,
                                   codebook=NONUNIFORM)
            cb = elem_bound(codes, X, xd, scales, sg, codebook=NONUNIFORM,   # (a problem this small: full-width tables)
                            table16=B.msgemm_plan_get_info(plan)["variant"] == B.VARIANT_FUSED_LDS16)
            check(run(lambda Y: B.msgemm_run(plan, dX, k, Y, m)), want, xd, "value map", cb)
            check(run(lambda Y: B.msgemm_run_static(plan, dX, k, Y, m)), want, xd, "value map, static", cb)
            B.msgemm_plan_set_codebook(plan, None)
            assert np.array_equal(run(lambda Y: B.msgemm_run(plan, dX, k, Y, m)), first)
        assert B.msgemm_plan_check(plan) == B.OK
    finally:
        B.msgemm_destroy(plan)


def test_plan_info_names_the_kernels_that_serve_a_value_map():
    """Nine columns and 8 MiB of codes: the table kernels for it have 16-bit entries.  With a value map installed the plan
    reports them, with their limits, and the matrix form again when the paper's map is back."""
    m, k, b = 4096, 4096, 9
    codes, X = inputs.make_codes(m, k, seed=31), inputs.make_x(k, b, "f16", seed=32)
    dX, Y = torch_io.to_device(X, "f16"), torch_io.empty_output(b, m, "f16")
    plan = B.msgemm_plan(m, k, b, "f16", "f16", 2, 0, torch_io.to_device(codes, "codes"))
    try:
        shape = ("variant", "tile_rows", "tile_groups", "split_k", "col_chunk")
        at_first = B.msgemm_plan_get_info(plan)
        assert matrix_form(at_first)
        beyond = list(NONUNIFORM)
        beyond[3] = 70000.0
        assert B.msgemm_plan_set_codebook(plan, beyond, check=False) == B.ERR_UNSUPPORTED
        assert [B.msgemm_plan_get_info(plan)[f] for f in shape] == [at_first[f] for f in shape]   # (nothing was installed)
        B.msgemm_plan_set_codebook(plan, NONUNIFORM)
        info = B.msgemm_plan_get_info(plan)
        assert info["variant"] == B.VARIANT_FUSED_LDS16 and info["col_chunk"] == 8 and info["tile_groups"] in (16, 32)
        B.msgemm_run(plan, dX, k, Y, m)
        torch.cuda.synchronize()
        check(torch_io.to_host(Y), oracle.gemm_f64(codes, X.astype(np.float64), codebook=NONUNIFORM), "f16", "value map",
              elem_bound(codes, X, "f16", None, 0, table16=True, codebook=NONUNIFORM))
        big = dX.clone()
        big[2, 5] = 60000.0                              # times a value of 6: outside the 16-bit entries
        B.msgemm_run(plan, big, k, Y, m)
        assert B.msgemm_plan_check(plan) == B.ERR_RANGE
        B.msgemm_plan_set_codebook(plan, None)
        assert [B.msgemm_plan_get_info(plan)[f] for f in shape] == [at_first[f] for f in shape]
    finally:
        B.msgemm_destroy(plan)


CUS = 256
CHOICES = [
    # m, k, b, xd, matrix form: the two sides of some of the lines of the library's own choice
    (32768, 1024, 1, "f32", True), (32896, 1024, 1, "f32", False),      # one fp32 column: 32 Mi weights
    (32896, 1024, 2, "f32", True),
    (2048, 12288, 1, "f32", True), (2048, 16084, 1, "f32", False),      # ... and long chains although k is cut
    (448, 8192, 1, "f32", True), (448, 12288, 16, "f32", True),         # (two and four segments)
    (240 * CUS, 128, 1, "f16", True), (240 * CUS + 1, 128, 1, "f16", False), (240 * CUS + 1, 258, 1, "f16", True),
    (512 * CUS, 512, 5, "f16", True), (512 * CUS + 1, 512, 5, "f16", False), (512 * CUS + 1, 514, 5, "f16", True),
    (200 * CUS, 64, 48, "f16", True), (200 * CUS + 1, 64, 48, "f16", False),    # (three passes over 16 columns)
    (117 * CUS + 1, 66, 48, "f16", True), (118 * CUS, 66, 48, "f16", False),
    (600 * CUS, 514, 1, "bf16", True), (600 * CUS + 1, 514, 1, "bf16", False), (600 * CUS + 1, 640, 1, "bf16", True),
    (1024 * CUS, 640, 1, "f16", True), (1024 * CUS + 1, 640, 1, "f16", False),
    (64, 256, 3, "f16", True),
]


@pytest.mark.parametrize("m,k,b,xd,matrix", CHOICES)
def test_where_the_matrix_form_is_the_librarys_own_choice(m, k, b, xd, matrix):
    if torch.cuda.get_device_properties(0).multi_processor_count != CUS:
        pytest.skip("the lines are in rows per compute unit")
    codes = torch.randint(0, 256, (m, k // 2), dtype=torch.uint8, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(m + k))
    X = inputs.make_x(k, b, xd, seed=3)
    plan = B.msgemm_plan(m, k, b, xd, Y_OF_X[xd], 2, 0, codes)
    try:
        info = B.msgemm_plan_get_info(plan)
        assert matrix_form(info) == matrix
        Y = torch_io.empty_output(b, m, Y_OF_X[xd])
        Y.fill_(-3)
        B.msgemm_run(plan, torch_io.to_device(X, xd), k, Y, m)
        torch.cuda.synchronize()
        out = torch_io.to_host(Y)
    finally:
        B.msgemm_destroy(plan)
    rows = np.unique(np.concatenate([np.arange(min(m, 70)), np.arange(m - min(m, 70), m), np.random.default_rng(m).integers(0, m, 60)]))
    some = np.ascontiguousarray(codes.cpu().numpy()[rows])
    check(np.ascontiguousarray(out[:, rows]), oracle_y(some, X, xd, None, 0), xd, "own choice",
          elem_bound(some, X, xd, None, 0, table16=info["variant"] == B.VARIANT_FUSED_LDS16))


def e5m2_values():
    """OCP E5M2 patterns (1 sign, 5 exponent bits with bias 15, 2 mantissa bits); infinities and NaNs are given numbers."""
    v = np.empty(256)
    for p in range(256):
        e, f = (p >> 2) & 31, p & 3
        v[p] = f * 2.0 ** -16 if e == 0 else (1 + f / 4) * 2.0 ** (e - 15)
        if e == 31:
            v[p] = [0.0, 1.5, 3.0, 57344.0][f]
        if p & 0x80:
            v[p] = -v[p]
    return v


@pytest.mark.parametrize("m,k,b,xd,sg,options", [
    (131, 1666, 1, "f16", 0, {}), (131, 1666, 4, "bf16", 0, {"panels_per_workgroup": 2}), (100, 640, 8, "f16", 128, {}),
    (100, 640, 16, "bf16", 128, {"panels_per_workgroup": 2}), (47, 130, 3, "f32", 0, {}), (47, 1154, 12, "f32", 0, {}),
    (64, 256, 20, "f16", 256, {}), (33, 126, 2, "f32", 0, {}), (70, 2560, 2, "f16", 128, {"batched_segments": 3})])
@pytest.mark.parametrize("table", ["e4m3", "e5m2", "other"])
def test_codes8_of_a_device_format(table, m, k, b, xd, sg, options):
    """8-bit weights whose value map is an 8-bit floating-point format times a power of two run in the matrix form; every
    pattern occurs, those without a number in the format with the values the map gives them.  Any other map keeps the tables."""
    values = {"e4m3": np.nan_to_num(inputs.fp8_e4m3_values(), nan=-0.5) / 16, "e5m2": e5m2_values() * 2.0 ** -12,
              "other": np.nan_to_num(inputs.fp8_e4m3_values(), nan=0.3) / 16}[table]
    codes = np.random.default_rng(m + k + b).integers(0, 256, size=(m, k), dtype=np.uint8)
    codes[0, :126] = np.arange(126) + 130   # (patterns up to 255, the specials among them)
    X = inputs.make_x(k, b, xd, seed=k + 1)
    scales = inputs.make_scales(m, k, sg, seed=10) if sg else None
    Xd = oracle.bf16_bits_to_f64(X) if xd == "bf16" else X.astype(np.float64)
    ref = oracle.gemm_f64_codes8(codes, Xd, values, scales, sg)
    plan = B.msgemm_plan_codes8(m, k, b, xd, Y_OF_X[xd], sg, torch_io.to_device(codes, "codes"),
                                torch_io.to_device(scales, "scales"), values, options=dict(options, batched_form=3))
    try:
        matrix = B.msgemm_plan_get_info(plan)["tile_groups"] == 128
        assert matrix == (table != "other")
        Y = torch_io.empty_output(b, m, Y_OF_X[xd], ldy=m + 1)
        Y.fill_(-3)
        B.msgemm_run(plan, torch_io.to_device(X, xd), k, Y, m + 1)
        torch.cuda.synchronize()
        out = torch_io.to_host(Y)
    finally:
        B.msgemm_destroy(plan)
    check(np.ascontiguousarray(out[:, :m]), ref, xd, f"8-bit weights {table}",
          elem_bound(codes, X, xd, scales, sg, table16=not matrix and b > 2 and xd != "f32", values256=values))


@pytest.mark.parametrize("xd,magnitude", [("bf16", 1e35), ("f32", 1e35), ("bf16", 1e-36), ("f32", 1e-36), ("f16", 1e4)])
@pytest.mark.parametrize("power", [-20, -12, 12, 19])
@pytest.mark.parametrize("b,sg,options", [(1, 0, {}), (12, 128, {}), (20, 0, {}), (2, 0, {"batched_segments": 3})])
def test_codes8_power_of_two_of_the_map_at_the_ends_of_the_range(b, sg, options, power, xd, magnitude):
    """The products are those of the map's own values: neither the format's (up to 57344 times as large) nor the power of two
    takes a sum out of the range of fp32 when the result is inside it, or under its smallest normal number."""
    if xd != "f16" and (power > 0) == (magnitude > 1):
        pytest.skip("results outside the range of fp32, or near its end")
    if power > 0 and b > 2 and xd != "f32":
        pytest.skip("refused: values over 65504 where the table kernels have 16-bit entries")
    m, k, two = 64, 1280 if sg else 1282, 2.0 ** power
    values = e5m2_values() * two
    codes = np.random.default_rng(m + b).integers(0, 256, size=(m, k), dtype=np.uint8)
    X = (inputs.make_x(k, b, "f32", seed=k + 1) * np.float32(magnitude)).astype(np.float32)
    X = {"f32": X, "bf16": inputs.f32_to_bf16_bits(X), "f16": np.clip(X, -6e4, 6e4).astype(np.float16)}[xd]
    scales = inputs.make_scales(m, k, sg, seed=10) if sg else None
    Xd = oracle.bf16_bits_to_f64(X) if xd == "bf16" else X.astype(np.float64)
    ref = oracle.gemm_f64_codes8(codes, Xd, values, scales, sg)
    plan = B.msgemm_plan_codes8(m, k, b, xd, Y_OF_X[xd], sg, torch_io.to_device(codes, "codes"),
                                torch_io.to_device(scales, "scales"), values, options=dict(options, batched_form=3))
    try:
        assert B.msgemm_plan_get_info(plan)["tile_groups"] == 128
        Y = torch_io.empty_output(b, m, Y_OF_X[xd])
        Y.fill_(-3)
        B.msgemm_run(plan, torch_io.to_device(X, xd), k, Y, m)
        torch.cuda.synchronize()
        out = torch_io.to_host(Y)
    finally:
        B.msgemm_destroy(plan)
    if xd == "f16" and np.abs(ref).max() > 6e4:
        over = np.abs(ref) > 65600                       # (outputs outside fp16: infinities of the right sign)
        assert np.array_equal(torch_io.to_f64(out)[over], np.inf * np.sign(ref[over]))
        return
    check(out, ref, xd, f"E5M2 times 2^{power}", elem_bound(codes, X, xd, scales, sg, values256=values))


@pytest.mark.parametrize("non_blocking", [1, 0])
def test_first_value_map_while_a_stream_is_captured(non_blocking):
    # the table kernels' plan is made at that point, outside the capture; the captured launch keeps the map it was given
    lib = B.load()  # (its symbols and those of the runtime it is linked to)
    m, k = 96, 512
    codes, X = inputs.make_codes(m, k, seed=21), inputs.make_x(k, 1, "f32", seed=22)
    dX, Y = torch_io.to_device(X, "f32"), torch.zeros((1, m), dtype=torch.float32, device="cuda:0")
    plan = B.msgemm_plan(m, k, 1, "f32", "f32", 2, 0, torch_io.to_device(codes, "codes"))
    B.msgemm_run(plan, dX, k, Y, m)
    torch.cuda.synchronize()
    stream, graph, instance = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    assert lib.hipStreamCreateWithFlags(ctypes.byref(stream), non_blocking) == 0
    assert lib.hipStreamBeginCapture(stream, 0) == 0  # (global mode)
    B.msgemm_plan_set_codebook(plan, NONUNIFORM)
    B.msgemm_run(plan, dX, k, Y, m, stream.value)
    assert lib.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0 and graph.value
    B.msgemm_plan_set_codebook(plan, None)
    assert lib.hipGraphInstantiate(ctypes.byref(instance), graph, None, None, ctypes.c_size_t(0)) == 0
    want = oracle.gemm_f64(codes, X.astype(np.float64), None, 0, codebook=NONUNIFORM)
    for _ in range(3):
        Y.zero_()
        torch.cuda.synchronize()
        assert lib.hipGraphLaunch(instance, stream) == 0 and lib.hipStreamSynchronize(stream) == 0
        assert oracle.rel_l2(torch_io.to_f64(torch_io.to_host(Y)), want) < 1e-5
    assert lib.hipGraphExecDestroy(instance) == 0 and lib.hipGraphDestroy(graph) == 0
    assert lib.hipStreamDestroy(stream) == 0
    B.msgemm_destroy(plan)


def _random_cases(count, seed):
    rng = np.random.default_rng(seed)
    cases = []
    while len(cases) < count:
        xd = ["f32", "f16", "bf16", "i8"][rng.integers(4)]
        m, k = int(rng.integers(1, 1500)), 2 * int(rng.integers(1, 1400))
        sg = 0 if xd == "i8" else int([0, 0, 128, 256, 384][rng.integers(5)])
        if sg:
            k = max(sg, (k // sg) * sg)
        b = int([1, 1, 2, 3, 4, 5, 8, 9, 13, 16, 17, 24, 32, 40, 48, 64, 70, 130][rng.integers(18)])
        options = [None, {"batched_form": 3}, {"batched_form": 3, "rows_per_lane": int([4, 8][rng.integers(2)])},
                   {"batched_form": 3, "panels_per_workgroup": int(rng.integers(1, 5))},
                   {"batched_form": 3, "batched_segments": int(rng.integers(2, 6)), "rows_per_lane": int([4, 8][rng.integers(2)])}]
        cases.append((m, k, b, xd, sg, options[rng.integers(5)]))
    return cases


@pytest.mark.parametrize("m,k,b,xd,sg,options", _random_cases(160, seed=23100617))
def test_random_shapes_in_the_matrix_form(m, k, b, xd, sg, options):
    """Seeded random problems by the library's own choice, which is the matrix form for all of them, and with requests for
    its kernels and shapes (those that do not fit the problem fall back to its choice)."""
    codes = inputs.make_codes(m, k, seed=m * 31 + k)
    X = inputs.make_x(k, b, xd, seed=k * 7 + b)
    scales = inputs.make_scales(m, k, sg, seed=m + b) if sg else None
    out, info = run_gpu(codes, X, xd, scales, sg, 0, B.VARIANT_AUTO, ldx_pad=2, ldy_pad=1, options=options)
    assert matrix_form(info)
    check(out, oracle_y(codes, X, xd, scales, sg), xd, f"{m}x{k}x{b} {xd} sg={sg} {options}", elem_bound(codes, X, xd, scales, sg))
