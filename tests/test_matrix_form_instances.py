"""Every instance of the matrix form's kernels (type, weights, row tiles, columns, wavefronts, ring depth, scales, direct loads or not), against the
CPU oracle: each problem here is the smallest that the library's rule gives to its instance.  That together they run all of them, and which
kernels the rule chooses, is checked without a GPU in test_matrix_form_choice.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_06178_amd import binding as B
from paper_2310_06178_amd import inputs, torch_io
from test_gpu_parity import Y_OF_X, check, elem_bound, oracle_y

pytestmark = pytest.mark.gpu

E4M3 = np.nan_to_num(inputs.fp8_e4m3_values(), nan=0.0) / 16
E5M2 = np.array([(1 - 2 * (p >> 7)) * ((p & 3) * 2.0 ** -16 if not p & 124 else (1 + (p & 3) / 4) * 2.0 ** ((p >> 2 & 31) - 15)) for p in range(256)])
E5M2 = np.where(np.arange(256) & 124 == 124, 0.25, E5M2) / 4096
MAPS = {"e4m3": E4M3, "e5m2": E5M2}
RUN = 128


def _cases():
    """(m, k, b, type of X, scale block, weights, options, distance of the columns of X or 0)"""
    cases = []

    def add(m, runs, b, x, scaled, weights="int4", ldx=0, **options):
        if scaled and x == "i8":
            return
        k = runs * RUN if scaled else runs * RUN + (16 if x == "i8" and runs == 97 else 2)   # (unscaled: a ragged run of a few columns behind the full ones)
        cases.append((m, k, b, x, RUN if scaled else 0, weights, dict(options, batched_form=3), ldx))

    for x in ("f16", "bf16", "f32", "i8"):
        for scaled in (False, True):
            for runs in (5, 17, 34):                     # one row tile: rings of two, of four, sixteen wavefronts
                add(33, runs, 1, x, scaled, panels_per_workgroup=1)
            if x != "f32":                               # ... eight wavefronts (int8: of whole 16-byte pieces)
                add(33, 161 if x == "bf16" and scaled else 97, 1, x, scaled, panels_per_workgroup=1, batched_segments=1)
            if x != "f32":
                add(33, 161, 3, x, scaled, panels_per_workgroup=1, batched_segments=1)      # ... rings of eight
            add(65, 9, 2, x, scaled, panels_per_workgroup=2)            # two and four row tiles
            add(130, 9, 4, x, scaled, panels_per_workgroup=4)
            # more than one workgroup a compute unit (256 of them): segments make them out of few rows
            segments = dict(panels_per_workgroup=2, batched_segments=8)
            if x == "i8":
                if not scaled:                           # ... a k of whole runs, and a long one that is none
                    cases.append((2070, 8 * 80 * RUN, 1, x, 0, "int4", dict(segments, batched_form=3), 0))
                for r in (1, 2):
                    add(70, 81, 13, x, scaled, panels_per_workgroup=r, batched_segments=1)
                add(1050, 8 * 3, 13, x, scaled, **segments)
            else:
                add(1050, 8 * 6, 3, x, scaled, **segments)
                if x != "f32":
                    add(1050, 8 * 28, 1, x, scaled, **segments)
            if x != "i8":
                for r in (1, 2, 4):                      # five to eight columns, one workgroup a compute unit and more
                    add(70, 17, 7, x, scaled, panels_per_workgroup=r)
                add(1050, 8 * 3, 5, x, scaled, **segments)
                if x == "f32":
                    for r in (1, 2, 4):
                        add(70, 3, 6, x, scaled, panels_per_workgroup=r)
            for r in (1, 2, 4):                          # nine to sixteen
                add(70, 17, 13, x, scaled, panels_per_workgroup=r)
                if x == "f32":
                    add(70, 3, 12, x, scaled, panels_per_workgroup=r)
            if x != "f32":
                add(70, 81, 20, x, scaled, panels_per_workgroup=2, rows_per_lane=8, batched_segments=1)     # two passes over a long k
                # four passes that fill the compute units (int8: of a k of whole runs)
                if x == "i8" and not scaled:
                    cases.append((3584, 17 * RUN, 60, x, 0, "int4", dict(panels_per_workgroup=4, rows_per_lane=8, batched_form=3), 0))
                else:
                    add(3584, 17, 60, x, scaled, panels_per_workgroup=4, rows_per_lane=8)
    for weights in MAPS:
        for x in ("f16", "bf16", "f32"):
            for scaled in (False, True):
                for r in (1, 2):
                    for b in (3, 8, 14):
                        add(70, 9, b, x, scaled, weights, panels_per_workgroup=r)
    # tile kernel: 17 to 32 columns and up to 64, with columns of X near each other and gigabytes apart
    for x in ("f16", "bf16", "i8"):
        for b in (21, 50):
            for r in (1, 2, 3):
                for weights in ("int4", "e4m3", "e5m2"):
                    for scaled in (False, True):
                        if (weights != "int4" and (x == "i8" or r == 3 or (scaled and b == 50 and r == 2))) or (scaled and r == 3):
                            continue
                        far = 2 ** 31 // ((33 if b < 33 else 65) * (1 if x == "i8" else 2)) + 3
                        for ldx in (0, far):
                            if x == "i8" and b == 21:    # (asked for, it would be the kernel of 16-row tiles)
                                add(11008, 8, b, x, scaled, weights, ldx, panels_per_workgroup=r)
                            else:
                                add(70, 5, b, x, scaled, weights, ldx, panels_per_workgroup=r, rows_per_lane=4)
    return cases


CASES = _cases()
# int8, 17 to 64 columns: the tile kernel of 16-row tiles over the lengths it is chosen for, rings that wrap, segments; and its own choice of the larger one
SMALL = [(m, runs * RUN + 2, b, "i8", 0, "int4", dict(o, batched_form=3, rows_per_lane=4, panels_per_workgroup=r), 0)
         for r in (1, 2, 3) for b in (17, 32, 33, 48) for m, runs, o in ((70, 27, {}), (200, 40, {"batched_segments": 2}))]
SMALL += [(m, runs * RUN + 2, b, "i8", 0, "int4", dict(o, batched_form=3, rows_per_lane=4, panels_per_workgroup=r), 0)
          for r in (1, 2, 3) for b in (49, 64) for m, runs, o in ((70, 67, {"batched_segments": 1}), (200, 133, {"batched_segments": 2}))]
SMALL += [(11008, 5126, 40, "i8", 0, "int4", None, 0), (33000, 130, 32, "i8", 0, "int4", None, 0), (33000, 386, 20, "i8", 0, "int4", None, 0)]
# the tile kernel by the library's own choice
OWN = [(4200, 14338, 40, "f16", 0, "int4", None, 0), (11008, 512, 64, "bf16", 128, "int4", None, 0), (16384, 130, 20, "f16", 0, "int4", None, 0),
       (11008, 1026, 20, "bf16", 0, "e4m3", None, 0)]


@pytest.mark.parametrize("m,k,b,x,group,weights,options,ldx", CASES + SMALL + OWN)
def test_against_oracle(m, k, b, x, group, weights, options, ldx):
    bits = 4 if weights == "int4" else 8
    codes = torch.randint(0, 256, (m, k * bits // 8), dtype=torch.uint8, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(m + k + b))
    X = inputs.make_x(k, b, x, seed=k + b)
    scales = inputs.make_scales(m, k, group, seed=6) if group else None
    dX, dS = torch_io.to_device(X, x), torch_io.to_device(scales, "scales")
    if ldx:
        small, dX = dX, torch.empty((b - 1) * ldx + k, dtype=dX.dtype, device="cuda:0")
        for c in range(b):
            dX[c * ldx:c * ldx + k] = small[c]
    if bits == 4:
        plan = B.msgemm_plan(m, k, b, x, Y_OF_X[x], 2, group, codes, dS, options=options)
    else:
        plan = B.msgemm_plan_codes8(m, k, b, x, Y_OF_X[x], group, codes, dS, MAPS[weights], options=options)
    try:
        Y = torch_io.empty_output(b, m, Y_OF_X[x], ldy=m + 5)
        Y.fill_(-3)
        B.msgemm_run(plan, dX, ldx or k, Y, m + 5)
        torch.cuda.synchronize()
        out = torch_io.to_host(Y)
    finally:
        B.msgemm_destroy(plan)
    assert np.all(torch_io.to_f64(out)[:, m:] == -3)
    rows = np.unique(np.concatenate([np.arange(min(m, 70)), np.arange(m - min(m, 70), m), np.random.default_rng(m).integers(0, m, 60)]))
    codes, out = np.ascontiguousarray(codes.cpu().numpy()[rows]), np.ascontiguousarray(out[:, :m][:, rows])
    scales = None if scales is None else np.ascontiguousarray(scales[rows])
    if bits == 4:
        ref, bound = oracle_y(codes, X, x, scales, group), elem_bound(codes, X, x, scales, group)
    else:
        Xd = oracle.bf16_bits_to_f64(X) if x == "bf16" else X.astype(np.float64)
        ref = oracle.gemm_f64_codes8(codes, Xd, MAPS[weights], scales, group)
        bound = elem_bound(codes, X, x, scales, group, values256=MAPS[weights])
    check(out, ref, x, f"{weights} {options}", bound)
