"""Which kernel of the matrix form a problem runs in, by the library's own choice, on the CPU: libmsgemm.so over a stand-in for the HIP runtime
(recording_hip_runtime.c, 256 compute units) that notes the kernels launched.  Problems on both sides of the lines of its rule."""
import json
import os
import re
import subprocess
import sys

import pytest

import test_matrix_form_depths
import test_matrix_form_instances
import test_matrix_form_tiles
from test_matrix_form_instances import MAPS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

BODY = """
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.rec_kernel.restype = rec.rec_name.restype = ctypes.c_char_p
from paper_2310_06178_amd import binding as B
B.load()
A, launched = 0x10000, []
problems, maps = json.load(sys.stdin)
for m, k, b, x, group, weights, options, ldx in problems:
    scales, y = A if group else None, "i32" if x == "i8" else x
    if weights in maps:
        plan = B.msgemm_plan_codes8(m, k, b, x, y, group, A, scales, maps[weights], options=options, stream=0)
    else:
        plan = B.msgemm_plan(m, k, b, x, y, 2, group, A, scales, options=options, stream=0)
    rec.rec_forget()
    B.msgemm_run(plan, A, ldx or k, A, m, stream=0)
    launched.append([rec.rec_kernel(i).decode() for i in range(rec.rec_count())])
    B.msgemm_destroy(plan)
json.dump([launched, [rec.rec_name(i).decode() for i in range(rec.rec_kernels())]], sys.stdout)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "librecording_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-Wextra", "-Werror", "-o", out,
                    os.path.join(ROOT, "tests", "recording_hip_runtime.c")], check=True)
    return out


def launches(runtime, problems):
    """Kernels that msgemm_run launches for each (m, k, b, x, scale group[, weights, options, ldx]), and all that the library has."""
    full = [list(p) + ["int4", None, 0][len(p) - 5:] for p in problems], {name: values.tolist() for name, values in MAPS.items()}
    p = subprocess.run([sys.executable, "-c", BODY, runtime], cwd=ROOT, input=json.dumps(full), capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-3000:]
    return json.loads(p.stdout)


def short(name):
    """stream R/W x D, tile R/column tiles, small R/column tiles, or tables."""
    ints = [int(i) for i in re.findall(r"L[ib](\d+)E", name)]
    if "matrix_stream_kernel" in name:
        return "stream %d/%dx%d" % (ints[0], ints[2], ints[3])
    if "matrix_tile_kernel" in name:
        return "tile %d/%d" % (ints[1], ints[2])
    if "matrix_small_tile_kernel" in name:
        return "small %d/%d" % (ints[0], ints[1])
    return "tables"


# m, k, b, type of X, scale block, kernel
CHOICES = [
    # int8, two row tiles: rings of four in four wavefronts, unless three workgroups and more have 80 runs and more each
    (14848, 10240, 1, "i8", 0, "stream 2/4x4"), (14848, 40192, 1, "i8", 0, "stream 2/4x4"), (19847, 6744, 4, "i8", 0, "stream 2/4x4"),
    (37725, 6744, 8, "i8", 0, "stream 2/4x4"), (32760, 9900, 1, "i8", 0, "stream 2/4x4"), (26000, 10240, 1, "i8", 0, "stream 2/8x2"),
    # 16 bits: one row tile where that takes the busiest compute unit fewer row tiles, and for one column under four workgroups a compute unit
    # or a short stream also where it takes as many
    (11008, 4860, 1, "f16", 0, "stream 1/4x2"), (18097, 8192, 2, "f16", 128, "stream 1/4x4"), (33280, 8192, 1, "bf16", 0, "stream 1/4x4"),
    (33280, 8192, 4, "bf16", 0, "stream 2/8x2"), (20480, 12288, 1, "f16", 0, "stream 2/8x2"),
    (16384, 4096, 1, "f16", 0, "stream 1/4x2"), (8192, 8192, 1, "bf16", 128, "stream 1/4x4"), (16400, 4096, 1, "f16", 0, "stream 1/4x2"),
    (24089, 5888, 1, "f16", 128, "stream 2/8x2"), (13160, 8192, 2, "f16", 128, "stream 2/8x2"), (24089, 4860, 4, "bf16", 0, "stream 2/8x2"),
    (24089, 2944, 4, "bf16", 0, "stream 1/4x2"), (7043, 2176, 3, "f16", 128, "stream 2/4x4"), (24089, 2944, 4, "f16", 128, "stream 2/4x2"), (24089, 2944, 1, "f16", 128, "stream 2/4x2"), (24089, 2944, 1, "f16", 0, "stream 1/4x2"),
    (33000, 2560, 2, "f16", 128, "stream 1/4x2"), (12759, 896, 4, "bf16", 128, "stream 1/4x2"), (40720, 1280, 4, "bf16", 256, "stream 2/4x4"), (46335, 1024, 2, "f16", 128, "stream 2/4x2"), (46335, 1536, 2, "f16", 128, "stream 2/4x4"), (24089, 1664, 2, "f16", 128, "stream 2/4x2"), (6056, 8192, 2, "f16", 0, "stream 2/4x4"),
    # a workgroup per compute unit: sixteen wavefronts from 32 runs on, eight from 92 on and where an unscaled k is whole turns of their rings, four
    # beyond 160 (fp16 with scales and more than two columns: 108); fp32, and bf16 with scales up to 160 or in two columns, sixteen
    (4096, 14336, 2, "f16", 128, "stream 1/8x4"), (4096, 11520, 2, "f16", 128, "stream 1/16x2"), (4096, 11776, 1, "bf16", 0, "stream 1/8x4"), (4096, 11648, 1, "bf16", 0, "stream 1/16x2"),
    (4096, 8192, 1, "f16", 0, "stream 1/8x4"), (4096, 8064, 1, "f16", 0, "stream 1/16x2"), (4096, 8192, 1, "f16", 128, "stream 1/16x2"), (4096, 3968, 1, "f16", 0, "stream 1/4x4"),
    (4096, 13696, 4, "f16", 128, "stream 1/8x4"), (4096, 13824, 4, "f16", 128, "stream 1/4x8"), (4096, 16384, 4, "f16", 128, "stream 1/4x8"),
    (4096, 20352, 4, "f16", 0, "stream 1/8x4"), (4096, 20480, 4, "f16", 0, "stream 1/4x8"), (3072, 40960, 3, "f16", 128, "stream 1/4x8"), (3072, 40960, 2, "f16", 128, "stream 1/8x4"),
    (3072, 24576, 2, "bf16", 128, "stream 1/16x2"), (3072, 24576, 1, "bf16", 128, "stream 1/8x4"), (3072, 20352, 3, "bf16", 128, "stream 1/16x2"), (3072, 20480, 3, "bf16", 128, "stream 1/4x8"),
    (4096, 40960, 4, "f32", 0, "stream 1/16x2"), (1792, 40960, 1, "f16", 0, "stream 1/4x8"),
    # int8 in few columns: sixteen wavefronts from 33 runs to 49, else eight from 26 runs up to 160 where columns are whole 16-byte pieces, and four with
    # rings of eight where they are not
    (4096, 4096, 1, "i8", 0, "stream 1/8x4"), (4096, 3328, 1, "i8", 0, "stream 1/8x4"), (4096, 4352, 2, "i8", 0, "stream 1/16x2"), (4096, 6400, 2, "i8", 0, "stream 1/8x4"),
    (4096, 20352, 4, "i8", 0, "stream 1/8x4"), (4096, 20480, 4, "i8", 0, "stream 1/4x8"), (2562, 15402, 4, "i8", 0, "stream 1/4x8"), (4096, 4100, 1, "i8", 0, "stream 1/16x2"),
    (4096, 4092, 1, "i8", 0, "stream 1/4x8"), (4096, 3844, 2, "i8", 0, "stream 1/4x8"), (4096, 6276, 1, "i8", 0, "stream 1/4x8"),
    (4096, 20480, 8, "i8", 0, "stream 1/4x8"), (4096, 4096, 8, "i8", 0, "stream 1/4x4"), (2562, 15402, 8, "i8", 0, "stream 1/4x8"),
    # a short k: rings of two up to ten runs; int8 in few columns keeps more in flight from 20 to 31 runs (25 in whole pieces), and under three workgroups where
    # columns end inside a 16-byte piece
    (3072, 1280, 1, "f16", 0, "stream 1/4x2"), (3072, 1290, 1, "f16", 0, "stream 1/4x4"), (3072, 1290, 8, "i8", 0, "stream 1/4x4"),
    (3072, 1290, 1, "f32", 0, "stream 1/4x2"), (3072, 2580, 1, "i8", 0, "stream 1/4x8"), (3072, 2820, 4, "i8", 0, "stream 1/4x8"),
    (3072, 3070, 1, "i8", 0, "stream 1/4x8"), (3072, 2178, 1, "i8", 0, "stream 1/4x4"), (3072, 2562, 4, "i8", 0, "stream 1/4x4"),
    (3072, 2816, 2, "i8", 0, "stream 1/4x8"), (3072, 2816, 8, "i8", 0, "stream 1/4x4"), (3072, 3330, 1, "i8", 0, "stream 1/4x8"), (512, 3686, 3, "i8", 0, "stream 1/4x8"), (3072, 3334, 4, "i8", 0, "stream 1/4x4"),
    (3072, 3596, 2, "i8", 0, "stream 1/4x8"), (12288, 3640, 1, "i8", 0, "stream 1/4x4"),
    (12288, 3648, 1, "i8", 0, "stream 1/4x2"), (12288, 4096, 1, "i8", 0, "stream 1/4x2"), (12288, 3640, 8, "i8", 0, "stream 1/4x2"),
    # more than 16 columns: tiles where they fill five eighths of the device or the passes' codes are 80 MiB, tables beyond 2400 rows a compute
    # unit of a single run; int8 up to 48 columns: the kernel of 16-row tiles from 20 runs on, up to
    # 64 from 66 on
    (10304, 512, 20, "f16", 0, "tile 1/1"), (10240, 512, 20, "f16", 0, "stream 2/8x2"), (4200, 14338, 40, "f16", 0, "tile 2/2"), (4200, 10498, 40, "f16", 0, "stream 4/8x2"),
    (2400 * 256, 128, 17, "bf16", 0, "tile 3/1"), (2400 * 256 + 1, 128, 17, "bf16", 0, "tables"), (2400 * 256 + 1, 256, 17, "f16", 0, "tile 3/1"),
    (28672, 4096, 24, "i8", 0, "small 2/2"), (28672, 4096, 49, "i8", 0, "tile 2/2"), (27648, 10752, 50, "i8", 0, "small 2/4"), (27648, 8450, 64, "i8", 0, "small 2/4"),
    (27648, 8320, 64, "i8", 0, "tile 2/2"), (36864, 10752, 80, "i8", 0, "small 3/4"), (16384, 14336, 80, "i8", 0, "tile 2/2"), (49152, 10752, 100, "i8", 0, "tile 3/2"), (16384, 10752, 64, "i8", 0, "tile 2/2"), (16384, 20480, 64, "i8", 0, "small 2/4"),
    (28672, 2432, 24, "i8", 0, "tile 2/1"),
    # four row tiles and 16 columns: four wavefronts from nine sixteenths of the compute units on (int8: seven eighths; two workgroups each where k is no whole number of runs), but not in
    # three passes and more over a long k (bf16 with scales: two), nor for fewer columns with scales over a longer one
    (5120, 5120, 24, "bf16", 128, "stream 4/8x2"), (5120, 4992, 24, "bf16", 128, "stream 4/4x2"), (5120, 5120, 24, "bf16", 0, "stream 4/4x2"), (5120, 5120, 24, "f16", 128, "stream 4/4x2"),
    (11776, 7680, 11, "f16", 128, "stream 4/8x2"), (11776, 7552, 11, "f16", 128, "stream 4/4x2"), (11776, 12800, 12, "f16", 128, "stream 4/4x2"), (11776, 12800, 11, "f16", 0, "stream 4/4x2"),
    (143 * 64, 4096, 16, "f16", 128, "stream 4/8x2"), (144 * 64, 4096, 16, "f16", 128, "stream 4/4x2"), (223 * 64, 4096, 16, "i8", 0, "stream 4/8x2"),
    (224 * 64, 4096, 16, "i8", 0, "stream 4/4x2"), (26000, 8192, 16, "i8", 0, "stream 4/4x2"), (26000, 3000, 16, "i8", 0, "stream 4/4x2"), (7970, 2720, 32, "i8", 0, "stream 4/8x2"),
    (8192, 4096, 32, "bf16", 0, "stream 4/4x2"), (4096, 4096, 64, "f16", 128, "stream 4/4x2"), (4096, 5376, 64, "f16", 128, "stream 4/8x2"),
    # fp16 in two passes of two row tiles: four wavefronts with rings of four from 80 runs on
    (4096, 14336, 20, "f16", 0, "stream 2/4x4"), (4096, 10240, 32, "f16", 128, "stream 2/4x4"), (4096, 10112, 32, "f16", 128, "stream 2/8x2"), (4096, 14336, 20, "bf16", 0, "stream 2/8x2"),
    # int8 over a long k that is no whole number of runs: four wavefronts with rings of four
    (4000, 11428, 16, "i8", 0, "stream 1/4x4"), (4000, 11392, 16, "i8", 0, "stream 1/8x2"), (4000, 10000, 16, "i8", 0, "stream 1/8x2"), (5608, 11426, 9, "i8", 0, "stream 2/4x4"),
    (22868, 18240, 4, "i8", 0, "stream 2/4x4"), (22868, 18304, 4, "i8", 0, "stream 2/8x2"),
    # int8 in two row tiles, two workgroups a compute unit and more: four wavefronts under 16 runs
    (9984, 1536, 24, "i8", 0, "stream 2/4x2"), (18176, 1920, 16, "i8", 0, "stream 2/4x2"), (18176, 2048, 16, "i8", 0, "stream 2/8x2"),
    # int8, 49 columns and more under few rows: tiles from 112 MiB of codes in all passes on
    (8192, 7168, 64, "i8", 0, "tile 1/2"), (8192, 7166, 64, "i8", 0, "stream 4/8x2"),
]


def test_own_choice(runtime):
    launched, _ = launches(runtime, [c[:5] for c in CHOICES])
    got = [c[:5] + (short(names[0]),) for c, names in zip(CHOICES, launched)]
    assert got == CHOICES


def test_every_instance_is_run_by_a_gpu_test(runtime):
    """All instances of the matrix form's kernels that the library holds are launched by a problem of test_matrix_form_instances.py."""
    cases = test_matrix_form_instances.CASES + test_matrix_form_instances.SMALL
    launched, names = launches(runtime, cases)
    assert all(run for run in launched)
    held = {n for n in names if re.search("matrix_(stream|tile|small_tile|reduce)_kernel", n)}
    assert len(held) > 250
    assert held - {n for run in launched for n in run} == set()


def test_what_the_gpu_tests_of_a_kernel_run(runtime):
    """The problems that are named after a kernel run in it."""
    tiles = [(m, k, b, x, group, "int4", dict(o, batched_form=3, rows_per_lane=4), 0) for m, k, b, x, group, o, _ in test_matrix_form_tiles.CASES]
    tiles += [(m, k, b, "i8", 0) for m, k, b in test_matrix_form_tiles.SHORT8]
    assert {short(run[0])[:4] for run in launches(runtime, tiles)[0]} == {"tile"}
    small = test_matrix_form_instances.SMALL
    got = [short(run[0]) for run in launches(runtime, small)[0]]
    assert got[:-3] == ["small %d/%d" % (c[6]["panels_per_workgroup"], (c[2] + 15) // 16) for c in small[:-3]] and got[-3:] == ["small 2/3", "tile 3/1", "tile 3/1"]
    assert {short(run[0])[:4] for run in launches(runtime, test_matrix_form_instances.OWN)[0]} == {"tile"}
    depths = [(m, k, b, x, group, "int4", dict(o, batched_form=3), 0) for m, k, b, x, group, o in test_matrix_form_depths.CASES]
    got = {short(run[0]) for run in launches(runtime, depths)[0]}
    assert got >= {"stream 1/16x2", "stream 1/4x4", "stream 1/4x8", "stream 1/4x2", "stream 2/4x4", "stream 4/4x2", "stream 1/8x2"}, got
