"""The streaming kernel of the matrix form in every number of wavefronts and depth of rings that its rule chooses, against the
CPU oracle: runs of 128 columns that leave wavefronts without one, with one more than their neighbours and with a ragged one."""
import numpy as np
import pytest

import oracle
from paper_2310_06178_amd import binding as B
from paper_2310_06178_amd import inputs
from test_gpu_parity import check, elem_bound, oracle_y, run_gpu

pytestmark = pytest.mark.gpu

CASES = [(m, k, b, xd, sg, o) for xd, b in (("f16", 1), ("bf16", 4), ("f32", 3), ("i8", 8)) for m, k, sg, o in [
    # a workgroup per compute unit: sixteen wavefronts from 32 runs on
    (33, 31 * 128 + 2, 0, {}), (33, 32 * 128, 128, {}), (17, 33 * 128 - 2, 0, {}), (40, 47 * 128 + 66, 0, {}), (16, 64 * 128, 256, {}),
    (20, 49 * 128, 128, {}), (50, 130 * 128 + 4, 0, {"batched_segments": 2}),
    # two workgroups (of 256 compute units) and more
    (4200, 17 * 128 + 2, 0, {}), (4099, 19 * 128, 128, {}), (8300, 16 * 128, 0, {}), (8250, 9 * 128 + 34, 0, {}),
    # two and four row tiles
    (8300, 5 * 128 + 2, 0, {"panels_per_workgroup": 2}), (300, 9 * 128, 128, {"panels_per_workgroup": 2}),
    (700, 11 * 128 + 2, 0, {"panels_per_workgroup": 4}), (130, 8 * 128, 128, {"panels_per_workgroup": 4})] if not (sg and xd == "i8")]
CASES += [(4200, 257 * 128 + 2, 1, "f16", 0, {"panels_per_workgroup": 1})]   # a long k under many rows
CASES += [(m, k, b, xd, sg, {"panels_per_workgroup": r}) for r in (1, 2, 4) for xd, b in (("f16", 6), ("bf16", 11), ("f32", 8), ("f32", 16), ("i8", 16))
          for m, k, sg in [(70, 17 * 128 + 2, 0), (131, 23 * 128, 128)] if not (sg and xd == "i8")]


@pytest.mark.parametrize("m,k,b,xd,sg,options", CASES)
def test_against_oracle(m, k, b, xd, sg, options):
    codes = inputs.make_codes(m, k, seed=m + 3 * k + b)
    X = inputs.make_x(k, b, xd, seed=k + b)
    scales = inputs.make_scales(m, k, sg, seed=6) if sg else None
    out, _ = run_gpu(codes, X, xd, scales, sg, 2, B.VARIANT_AUTO, ldx_pad=3, ldy_pad=5, options=dict(options, batched_form=3))
    check(out, oracle_y(codes, X, xd, scales, sg), xd, f"{options}", elem_bound(codes, X, xd, scales, sg))


@pytest.mark.parametrize("b", [1, 4, 8, 16])
@pytest.mark.parametrize("magnitude", [1e-36, 1e37])
def test_fp32_activations_of_any_magnitude_and_an_infinity(b, magnitude):
    """The part that goes over a wavefront's runs again, with sixteen and eight wavefronts and a ragged run."""
    m, k = 40, 35 * 128 + 2
    codes = inputs.make_codes(m, k, seed=4)
    X = (inputs.make_x(k, b, "f32", seed=5) * np.float32(magnitude if magnitude < 1 else magnitude / 64)).astype(np.float32)
    out, _ = run_gpu(codes, X, "f32", None, 0, 2, B.VARIANT_AUTO, options={"batched_form": 3})
    # (results that are subnormal themselves: every rounding of a sum may be half a step, k / 32 + 16 of them)
    bound = elem_bound(codes, X, "f32", None, 0) + (k // 32 + 16) * 2.0 ** -150
    check(out, oracle_y(codes, X, "f32", None, 0), "f32", f"magnitude {magnitude}", bound)
    X[b - 1, k - 2] = np.inf
    out, _ = run_gpu(codes, X, "f32", None, 0, 2, B.VARIANT_AUTO, options={"batched_form": 3})
    v = np.array([oracle.decode(int(c)) for c in codes[:, (k - 2) // 2] & 15], dtype=np.float64)
    assert np.array_equal(np.isnan(out[-1]), v == 0) and np.all(out[-1][v != 0] == np.inf * v[v != 0])
    if b > 1:
        check(np.ascontiguousarray(out[:-1]), oracle_y(codes, X[:-1], "f32", None, 0), "f32", "other columns", bound[:-1])
