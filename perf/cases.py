"""What a user of this library has it do, as cases that can be timed: Y = M x X for int4 (and 8-bit) weight matrices,
through msgemm_plan / msgemm_plan_codes8 once and msgemm_run on every pass.

A pass is one call on one weight matrix, or -- for the short GeMVs and small batches of a decoding model -- one step
through a stack of weight matrices of the same shape, captured once in a HIP graph and replayed, as a serving loop does
it (and as bench.py launches its steps).  A stack's weights are several times what stays in the caches, like a model's.

Shapes: the benchmark's configurations, the paper's two GeMMs (12288 x 49152 and 49152 x 12288), and generic ones of
the same range with odd and ragged sizes.  Weight codes are uniform over all bit patterns, activations N(0, 1) (bf16
with one in a hundred ten times as large; int8 uniform), scales uniform over [0.005, 0.02].
"""
import math

import torch

from paper_2310_06178_amd import binding as B
from paper_2310_06178_amd import inputs

DEVICE = "cuda:0"
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8, "i32": torch.int32}
Y_OF_X = {"f32": "f32", "f16": "f16", "bf16": "bf16", "i8": "i32"}
BYTES = {"f32": 4, "f16": 2, "bf16": 2, "i8": 1, "i32": 4}

STACK_BYTES = 256 << 20  # weights that a stack of layers goes through in one pass, about
MOST_LAYERS = 8
MOST_WEIGHTS = 49152 * 12288       # the paper's matrices
MOST_MACS = MOST_WEIGHTS * 64


def _case(m, k, b, x, scale_group=0, bits=4, layers=1):
    return {"m": m, "k": k, "b": b, "x": x, "scale_group": scale_group, "bits": bits, "layers": layers}


def listed():
    return [
        # the smallest call: one projection of a small model, alone, launched from Python without a graph
        dict(_case(1024, 1024, 1, "f32"), name="single_1024_f32"),
        # decoding one token: the benchmark's default GeMV, eight layers of it
        dict(_case(16384, 4096, 1, "f16", layers=8), name="decode_16384x4096_f16"),
        # the same with shared scales and bf16, square
        dict(_case(8192, 8192, 1, "bf16", 128, layers=8), name="decode_8192_bf16_scaled"),
        # sizes that are no multiple of anything
        dict(_case(11003, 4098, 1, "f16", layers=8), name="decode_11003x4098_f16"),
        # two sequences at once, a long inner dimension (the down projection of an MLP)
        dict(_case(4096, 14336, 2, "f16", 128, layers=8), name="pair_4096x14336_f16_scaled"),
        # one token through the paper's first MLP matrix: 300 MB of codes in one call
        dict(_case(12288, 49152, 1, "f16"), name="single_12288x49152_f16"),
        # 8-bit floating-point weights (E4M3), one token
        dict(_case(8192, 8192, 1, "f16", 128, bits=8, layers=4), name="decode_fp8_8192_f16_scaled"),
        # full-precision activations, a handful of sequences
        dict(_case(4096, 4096, 4, "f32", layers=8), name="batch4_4096_f32"),
        # batched decoding with shared scales
        dict(_case(14336, 4096, 16, "f16", 128, layers=8), name="batch16_14336x4096_f16_scaled"),
        # int8 activations, whole-number results
        dict(_case(8192, 8192, 16, "i8", layers=8), name="batch16_8192_i8"),
        # a large batch (or a short prompt), bf16 with outliers and shared scales
        dict(_case(28672, 8192, 64, "bf16", 128), name="batch64_28672x8192_bf16_scaled"),
        # the same through the paper's second MLP matrix
        dict(_case(49152, 12288, 64, "f16"), name="batch64_49152x12288_f16"),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        x = rng.choice(["f16", "f16", "bf16", "bf16", "f32", "i8"])
        bits = 8 if x in ("f16", "bf16") and rng.random() < 0.15 else 4
        b = rng.choice([1, 1, 1, 2, 3, 4, 6, 8, 11, 16, 16, 24, 32, 47, 64])
        if x == "f32":
            b = min(b, 8)
        m, k = size(768, 49152), 2 * size(384, 24576)
        scale_group = 0 if x == "i8" else rng.choice([0, 128, 128, 256])
        if rng.random() < 0.5:  # half of the matrices have round sizes, as most models' have
            m, k = -(-m // 256) * 256, -(-k // 256) * 256
        elif scale_group:
            k = -(-k // scale_group) * scale_group
        if m * k * bits // 4 > MOST_WEIGHTS or m * k * b * (2 if x == "f32" else 1) > MOST_MACS:
            continue
        layers = max(1, min(MOST_LAYERS, STACK_BYTES // (m * k * bits // 8)))
        if m * k * b > 1 << 30:
            layers = 1
        return _case(m, k, b, x, scale_group, bits, layers)


def _values256():
    v = inputs.fp8_e4m3_values()
    return [0.0 if math.isnan(a) else float(a) for a in v]


def _weights(case, seed, layer):
    """Codes [m][k * bits / 8] and scales (or None) of one layer, on the GPU, from the seed alone."""
    g = torch.Generator(device=DEVICE).manual_seed(seed * 64 + layer)
    m, k = case["m"], case["k"]
    codes = torch.randint(0, 256, (m, k * case["bits"] // 8), dtype=torch.uint8, device=DEVICE, generator=g)
    if case["bits"] == 8:  # the two patterns that stand for NaN in E4M3 do not occur
        codes = torch.where((codes & 0x7F) == 0x7F, codes - 1, codes)
    scales = None
    if case["scale_group"]:
        scales = torch.rand((m, k // case["scale_group"]), device=DEVICE, generator=g) * 0.015 + 0.005
        scales = scales.to(torch.float16)
    return codes, scales


def _activations(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(seed * 64 + 63)
    shape = (case["b"], case["k"])
    if case["x"] == "i8":
        return torch.randint(-128, 128, shape, dtype=torch.int8, device=DEVICE, generator=g)
    x = torch.randn(shape, device=DEVICE, generator=g)
    if case["x"] == "bf16":
        x = torch.where(torch.rand(shape, device=DEVICE, generator=g) < 0.01, 10.0 * x, x)
    return x.to(TORCH[case["x"]])


class _Stack:
    """What a program keeps: a plan per weight matrix, the buffers, and the graph of a step if it has several."""

    def __init__(self, case, seed):
        self.m, self.k = case["m"], case["k"]
        yd = Y_OF_X[case["x"]]
        self.plans = []
        for layer in range(case["layers"]):
            codes, scales = _weights(case, seed, layer)
            if case["bits"] == 8:
                plan = B.msgemm_plan_codes8(self.m, self.k, case["b"], case["x"], yd, case["scale_group"], codes, scales,
                                            _values256())
            else:
                plan = B.msgemm_plan(self.m, self.k, case["b"], case["x"], yd, 2, case["scale_group"], codes, scales)
            self.plans.append(plan)
        self.x = _activations(case, seed)
        self.y = [torch.empty((case["b"], self.m), dtype=TORCH[yd], device=DEVICE) for _ in self.plans]
        torch.cuda.synchronize()  # the plans have read the codes and scales
        self.graph = None
        if len(self.plans) > 1:
            self.step()
            torch.cuda.synchronize()
            self.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(self.graph):
                self.step()

    def step(self):
        for plan, y in zip(self.plans, self.y):
            B.msgemm_run(plan, self.x, self.k, y, self.m)

    def __del__(self):
        self.graph = None
        for plan in getattr(self, "plans", []):
            B.msgemm_destroy(plan)


def prepare(case, seed):
    return _Stack(case, seed)


def run(state):
    if state.graph is not None:
        state.graph.replay()
    else:
        state.step()
    return state.y


def work(case):
    m, k, b, n = case["m"], case["k"], case["b"], case["layers"]
    per_layer = m * k * case["bits"] // 8 + m * b * BYTES[Y_OF_X[case["x"]]]
    if case["scale_group"]:
        per_layer += m * (k // case["scale_group"]) * 2
    return {"bytes": n * per_layer + k * b * BYTES[case["x"]], "flops": 2 * m * k * b * n}


def tolerance(case):
    """About four times what the path is off its 64-bit value: for 16-bit outputs their own rounding (2.1e-4 in fp16,
    1.7e-3 in bf16, relative 2-norm) and, with 16-bit table entries, those entries' (up to 3.4e-4); 32-bit sums over up to
    49152 terms for fp32; whole numbers are the same."""
    if case["x"] == "i8":
        return "exact"
    return {"f32": {"rel": 2e-6, "max": 4e-5}, "f16": {"rel": 1.5e-3, "max": 1e-2}, "bf16": {"rel": 7e-3, "max": 4e-2}}[case["x"]]


def exact(case, seed):
    """The direct sum in 64 bits, from the same codes, scales and activations; whole-number results need none."""
    if case["x"] == "i8":
        return None
    x = _activations(case, seed).double()
    if case["bits"] == 8:
        values = torch.tensor(_values256(), dtype=torch.float64, device=DEVICE)
    else:
        values = torch.tensor([i if i < 8 else i - 16 for i in range(16)], dtype=torch.float64, device=DEVICE)
    sg = case["scale_group"]
    out = []
    for layer in range(case["layers"]):
        codes, scales = _weights(case, seed, layer)
        y = torch.empty((case["b"], case["m"]), dtype=torch.float64, device=DEVICE)
        rows = max(1, (1 << 27) // case["k"])
        for r in range(0, case["m"], rows):
            c = codes[r:r + rows]
            if case["bits"] == 4:
                c = torch.stack([c & 15, c >> 4], dim=2).reshape(c.shape[0], -1)
            w = values[c.int()]
            if sg:
                w = w * scales[r:r + rows].double().repeat_interleave(sg, dim=1)
            y[:, r:r + rows] = (w @ x.t().contiguous()).t()
        out.append(y)
    return out
