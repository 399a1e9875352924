"""Which device and stream the host side of the library uses, and what it chooses, on the CPU: libmsgemm.so over a stand-in for the HIP runtime
(recording_hip_runtime.c) that knows several devices and computes nothing.  Each case runs in a process of its own."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ALLOC, LAUNCH, WORK, EVENT = 1, 2, 3, 4

PRELUDE = """
import ctypes, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2310_06178_amd import binding as B
lib = B.load()
device = ctypes.c_int()
def current():
    rec.hipGetDevice(ctypes.byref(device))
    return device.value
def calls(since):
    return [(rec.rec_kind(i), rec.rec_device(i), rec.rec_own_stream(i)) for i in range(since, rec.rec_count())]
ADDRESS = 0x10000
MAP = [0.0, 0.5] + [0.25 * i for i in range(14)]
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "librecording_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-Wextra", "-Werror", "-o", out,
                    os.path.join(ROOT, "tests", "recording_hip_runtime.c")], check=True)
    return out


def run(runtime, body):
    p = subprocess.run([sys.executable, "-c", PRELUDE + body, runtime], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stderr[-3000:]
    return p.stdout


def test_first_value_map_works_on_the_plans_device(runtime):
    """The table kernels' plan is allocated and filled on the device of the plan, whatever device is current, and the
    current device is the caller's again afterwards."""
    out = run(runtime, """
rec.hipSetDevice(2)
plan = B.msgemm_plan(96, 512, 1, "f16", "f16", 2, 128, ADDRESS, ADDRESS, stream=0)
made = calls(0)
assert made and all(d == 2 for _, d, _ in made)
rec.hipSetDevice(1)
since = rec.rec_count()
B.msgemm_plan_set_codebook(plan, MAP)
used = calls(since)
assert [k for k, _, _ in used].count(1) >= 3 and [k for k, _, _ in used].count(2) >= 2, used   # allocations and launches
assert all(d == 2 for _, d, _ in used), used
assert current() == 1
since = rec.rec_count()
B.msgemm_plan_set_codebook(plan, MAP[::-1])             # the next map: host only
B.msgemm_plan_set_codebook(plan, None)
assert rec.rec_count() == since and current() == 1
print("ok")
""")
    assert out.strip().endswith("ok")


def test_dispatch_order_is_not_looked_at_from_a_temporary_stream(runtime):
    """While a stream that waits for the null stream is captured, the table kernels' plan is made on a stream of its own; the
    look at how the device deals workgroups over its dies, made once per process, waits for a plan on the caller's stream."""
    out = run(runtime, """
m, k, b = 4096, 4096, 9                                  # (served by the batched table kernels)
plan = B.msgemm_plan(m, k, b, "f16", "f16", 2, 0, ADDRESS, stream=0)
rec.rec_capture(1)
since = rec.rec_count()
B.msgemm_plan_set_codebook(plan, MAP)
rec.rec_capture(0)
used = calls(since)
on_own = [kind for kind, _, own in used if own]
assert 2 in on_own and not [1 for kind, _, own in used if kind in (2, 3) and not own], used
since = rec.rec_count()
B.msgemm_plan(m, k, b, "f16", "f16", 2, 0, ADDRESS, None, B.VARIANT_FUSED_LDS16, stream=0)
first = calls(since)
since = rec.rec_count()
B.msgemm_plan(m, k, b, "f16", "f16", 2, 0, ADDRESS, None, B.VARIANT_FUSED_LDS16, stream=0)
assert len(first) > len(calls(since)), (first, calls(since))   # the look itself: here, and once
print("ok")
""")
    assert out.strip().endswith("ok")


def test_plans_of_8_bit_codes_make_no_event(runtime):
    """The event orders the making of the table kernels' plan behind the repack; 8-bit codes keep their map."""
    out = run(runtime, """
from paper_2310_06178_amd import inputs
values = [0.0 if v != v else float(v) for v in inputs.fp8_e4m3_values()]
eight = B.msgemm_plan_codes8(96, 512, 1, "f16", "f16", 0, ADDRESS, None, values, stream=0)
assert B.msgemm_plan_get_info(eight)["tile_groups"] == 128   # (the matrix form)
assert 4 not in [k for k, _, _ in calls(0)]
B.msgemm_plan(96, 512, 1, "f16", "f16", 2, 0, ADDRESS, stream=0)
assert [k for k, _, _ in calls(0)].count(4) == 1
print("ok")
""")
    assert out.strip().endswith("ok")


def test_the_matrix_form_serves_what_the_table_kernels_refuse(runtime):
    """Where a short k under many rows belongs to the tables but their partial sums would pass 2 GiB."""
    out = run(runtime, """
from paper_2310_06178_amd import inputs
values = [0.0 if v != v else float(v) for v in inputs.fp8_e4m3_values()]
for m, matrix in ((1 << 20, False), (1 << 22, True)):
    plan = B.msgemm_plan(m, 64, 200, "f16", "f16", 2, 0, ADDRESS, stream=0)
    info = B.msgemm_plan_get_info(plan)
    assert (info["variant"] == B.VARIANT_FUSED_LDS and info["tile_groups"] == 64) == matrix, info
    plan = B.msgemm_plan_codes8(m, 64, 200, "f16", "f16", 0, ADDRESS, None, values, stream=0)
    assert (B.msgemm_plan_get_info(plan)["tile_groups"] == 128) == matrix
print("ok")
""")
    assert out.strip().endswith("ok")


@pytest.mark.parametrize("group", [2, 8, 16, 30])
def test_scale_blocks_smaller_than_a_table_tile(runtime, group):
    """Scale blocks under 32 columns fit no k-tile of the tables in LDS: AUTO keeps its tables in device memory, a request for the
    batched kernel is refused, and so are 8-bit codes (whose tables are in LDS only)."""
    out = run(runtime, f"""
from paper_2310_06178_amd import inputs
values = [0.0 if v != v else float(v) for v in inputs.fp8_e4m3_values()]
for b in (3, 16, 48):
    for x in ("f16", "bf16"):
        plan = B.msgemm_plan(64, 4 * {group}, b, x, x, 2, {group}, ADDRESS, ADDRESS, stream=0)
        assert B.msgemm_plan_get_info(plan)["variant"] == B.VARIANT_GLOBAL_LUT
        for make in (lambda: B.msgemm_plan(64, 4 * {group}, b, x, x, 2, {group}, ADDRESS, ADDRESS, B.VARIANT_FUSED_LDS16, stream=0),
                     lambda: B.msgemm_plan_codes8(64, 2 * {group}, b, x, x, {group} // 2, ADDRESS, ADDRESS, values, stream=0)):
            try:
                make()
                raise SystemExit("accepted")
            except B.MsgemmError as e:
                assert e.status == B.ERR_UNSUPPORTED, e
print("ok")
""")
    assert out.strip().endswith("ok")
