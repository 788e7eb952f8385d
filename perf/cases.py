"""What is timed when the library is made faster: calls and call sequences of the public entry points
(paper_2509_09679_amd.binding, paper_2509_09679_amd.calibration) at the sizes they are used with.

A case is a dict of plain values.  "op" says what one pass does:

    quant      fused forward transform + quantisation (bq_butterfly_fwd_quant)
    transform  forward or inverse transform (bq_butterfly_fwd / bq_butterfly_inv)
    roundtrip  forward, inverse of its result, fused quantisation: the three calls a small model makes per layer
    fakequant  fake-quantised forward with the code-bin counts (bq_butterfly_fwd_fakequant)
    step       what one SGD step on the angles asks of the library: plan from the new angles, forward, backward
    backward   dx and dtheta of one batch (bq_butterfly_bwd)
    composite  transform of a width that is not a power of two (bq_kron_fwd / bq_kron_inv)
    calibrate  loss and gradient of one linear layer (ButterflyCalibrator.loss_and_grad)

Sizes come from the benchmark's workloads and from the tests' sweeps.
"""
import math

import torch

from paper_2509_09679_amd import binding as B
from paper_2509_09679_amd.calibration import ButterflyCalibrator, QuantSpec

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # decoding, one token in flight: nothing but latency
        dict(name="decode", op="quant", n=4096, heads=1, rows=1, dtype="f16", bits=4, group=128, scale="f16"),
        # decoding, a batch of sequences of a wider model
        dict(name="decode_batch", op="quant", n=8192, heads=1, rows=37, dtype="bf16", bits=4, group=128, scale="f16"),
        # one prompt, of a length that divides nothing
        dict(name="prompt", op="quant", n=4096, heads=1, rows=1777, dtype="f16", bits=4, group=128, scale="f16"),
        # the benchmark's calibration / prefill batch: 128 sequences of 2048 tokens, INT2
        dict(name="prefill", op="quant", n=4096, heads=1, rows=262144, dtype="f16", bits=2, group=128, scale="f16"),
        # the benchmark's small workload: per-token INT4 of narrow float32 rows, forward and back
        dict(name="narrow_f32", op="roundtrip", n=128, heads=1, rows=1024, dtype="f32", bits=4, group=128, scale="f32"),
        # per-head rotation of keys / queries, the benchmark's workload
        dict(name="per_head", op="quant", n=128, heads=32, rows=8192, dtype="bf16", bits=4, group=128, scale="f32"),
        # per-head rotation of a model whose width is not a power of two
        dict(name="per_head_12", op="transform", inverse=False, n=64, heads=12, rows=20011, dtype="f16"),
        # undoing a rotation on float32 rows of a middle size, odd batch
        dict(name="inverse_f32", op="transform", inverse=True, n=2048, heads=1, rows=40001, dtype="f32"),
        # the benchmark's backward batch
        dict(name="backward", op="backward", n=8192, heads=1, rows=65536, dtype="bf16"),
        # one SGD step on one sequence
        dict(name="step", op="step", n=4096, heads=1, rows=2048, dtype="f16"),
        # the benchmark's calibration of one layer, W2A4
        dict(name="calibrate", op="calibrate", n=4096, m=4096, rows=16384, dtype="f16", bits=4, group=128, wbits=2,
             wgroup=128, scale="f16"),
        # width 5120 = 40 x 128
        dict(name="composite", op="composite", inverse=False, d1=40, n=128, rows=10007, dtype="f16"),
    ]


def _log_int(rng, lo, hi):
    """An integer between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    op = rng.choice(["quant", "quant", "quant", "transform", "transform", "roundtrip", "fakequant", "step", "backward",
                     "composite", "calibrate"])
    dtype = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
    c = dict(op=op, dtype=dtype)
    if op == "calibrate":
        n = rng.choice([1024, 2048, 4096])
        c.update(n=n, m=_log_int(rng, 512, 4096), rows=_log_int(rng, 1024, 16384), dtype=rng.choice(["f16", "f16", "bf16"]),
                 bits=4, group=rng.choice([64, 128, n]), wbits=rng.choice([2, 4]), wgroup=rng.choice([64, 128]), scale="f16")
        return c
    if op == "composite":
        d1, n = rng.choice([3, 5, 7, 12, 20, 24, 37, 40]), rng.choice([64, 128, 128, 256])
        c.update(inverse=rng.random() < 0.5, d1=d1, n=n, rows=_log_int(rng, 16, (1 << 26) // (d1 * n)))
        return c
    if op in ("step", "backward"):
        n, heads = rng.choice([(4096, 1), (4096, 1), (8192, 1), (2048, 1), (1024, 2), (128, 32), (64, 12)])
        most = 1 << (28 if op == "backward" else 25)
    else:
        n, heads = rng.choice([(4096, 1), (4096, 1), (4096, 1), (8192, 1), (8192, 1), (2048, 1), (1024, 1), (512, 8), (128, 1),
                               (128, 32), (128, 40), (128, 12), (64, 12), (64, 24), (128, 5), (32, 3), (16384, 1)])
        most = 1 << (22 if op == "roundtrip" else 26 if n == 16384 else 28)
    c.update(n=n, heads=heads, rows=_log_int(rng, 1, most // (n * heads) // (2 if dtype == "f32" else 1)))
    if op == "transform":
        c.update(inverse=rng.random() < 0.5)
    if op in ("quant", "roundtrip", "fakequant"):
        c.update(bits=rng.choice([2, 4]), group=rng.choice([g for g in (32, 64, 128, 128, 256, n) if g <= n]),
                 scale=rng.choice(["f16", "f16", "f32"]))
    return c


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _heavy(gen, rows, width, dtype, outliers=True):
    """Student-t(3) rows with one per cent of the channels a hundred times larger, as activations have."""
    out = torch.empty((rows, width), dtype=DTYPES[dtype], device=DEV)
    gain = torch.ones(width, device=DEV)
    if outliers:
        pick = torch.randperm(width, generator=gen, device=DEV)[: max(1, width // 100)]
        gain[pick] = 100.0 if width >= 1024 else 30.0
    chunk = max(1, (1 << 25) // width)
    for r in range(0, rows, chunk):
        k = min(chunk, rows - r)
        z = torch.randn((k, width), generator=gen, device=DEV)
        c = torch.randn((k, width), generator=gen, device=DEV).square_()
        for _ in range(2):
            c += torch.randn((k, width), generator=gen, device=DEV).square_()
        z *= gain / (c / 3.0).sqrt_()
        out[r:r + k] = z.clamp_(-65504.0, 65504.0)
    return out


def _normal(gen, rows, width, dtype, std=1.0):
    out = torch.empty((rows, width), dtype=DTYPES[dtype], device=DEV)
    chunk = max(1, (1 << 26) // width)
    for r in range(0, rows, chunk):
        k = min(chunk, rows - r)
        out[r:r + k] = torch.randn((k, width), generator=gen, device=DEV) * std
    return out


def _angles(gen, n, heads):
    """U[-pi, pi), as in the benchmark's workloads."""
    k = n.bit_length() - 1
    return (torch.rand((heads, k, n // 2), generator=gen, device=DEV) * 2.0 - 1.0) * math.pi


def prepare(case, seed):
    gen = _generator(seed)
    op, n, rows, dtype = case["op"], case["n"], case["rows"], case["dtype"]
    s = dict(case)
    if op == "calibrate":
        W = _normal(gen, case["m"], n, dtype, 0.02)
        theta = 0.1 * _angles(gen, n, 1)
        s["cal"] = ButterflyCalibrator(W, QuantSpec(case["bits"], case["group"], case["scale"]),
                                       QuantSpec(case["wbits"], case["wgroup"], case["scale"]), theta=theta)
        s["x"] = _heavy(gen, rows, n, dtype)
        return s
    if op == "composite":
        d1 = case["d1"]
        s["plan"] = B.alloc_plan(_angles(gen, n, 1), n, 1)
        s["q1"] = torch.empty((d1, d1), dtype=torch.float32, device=DEV)
        B.bq_cayley_build(torch.randn(d1 * (d1 - 1) // 2, generator=gen, device=DEV) * 0.3, d1, s["q1"])
        s["x"] = _heavy(gen, rows, d1 * n, dtype)
        s["y"] = torch.empty_like(s["x"])
        s["desc"] = B.make_kron_rows(s["x"], n)
        return s
    heads = case["heads"]
    theta = _angles(gen, n, heads)
    x = _heavy(gen, rows, n * heads, dtype, outliers=op not in ("backward", "step"))
    s.update(x=x, theta=theta, plan=B.alloc_plan(theta, n, heads), desc=B.make_rows(x, n, heads))
    if op in ("transform", "roundtrip", "step", "fakequant"):
        s["y"] = torch.empty_like(x)
    if op == "roundtrip":
        s["back"] = torch.empty_like(x)
    if op in ("quant", "roundtrip"):
        s["codes"], s["scales"] = B.alloc_quant_outputs(rows, n, heads, case["bits"], case["group"], case["scale"], DEV)
    if op in ("quant", "roundtrip", "fakequant"):
        s["spec"] = B.make_quant(case["bits"], case["group"], case["scale"])
    if op == "fakequant":
        s["hist"] = torch.zeros(1 << case["bits"], dtype=torch.int64, device=DEV)
    if op in ("backward", "step"):
        s["dy"] = _normal(gen, rows, n * heads, dtype)
        s["dx"] = torch.empty_like(x)
        s["dtheta"] = torch.empty_like(theta)
        s["work"] = torch.empty(max(256, B.bq_butterfly_bwd_workspace_bytes(s["desc"])), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    op = s["op"]
    if op == "quant":
        B.bq_butterfly_fwd_quant(s["x"], s["plan"], s["codes"], s["scales"], s["spec"], s["desc"])
        return {"codes": s["codes"], "scales": s["scales"]}
    if op == "transform":
        (B.bq_butterfly_inv if s["inverse"] else B.bq_butterfly_fwd)(s["x"], s["y"], s["plan"], s["desc"])
        return s["y"]
    if op == "roundtrip":
        B.bq_butterfly_fwd(s["x"], s["y"], s["plan"], s["desc"])
        B.bq_butterfly_inv(s["y"], s["back"], s["plan"], s["desc"])
        B.bq_butterfly_fwd_quant(s["x"], s["plan"], s["codes"], s["scales"], s["spec"], s["desc"])
        return {"y": s["y"], "back": s["back"], "codes": s["codes"], "scales": s["scales"]}
    if op == "fakequant":
        B.bq_butterfly_fwd_fakequant(s["x"], s["plan"], s["y"], s["hist"], s["spec"], s["desc"])
        return {"yq": s["y"], "occupancy": s["hist"] / s["x"].numel()}
    if op == "step":
        B.bq_plan_build(s["theta"], s["n"], s["heads"], s["plan"])
        B.bq_butterfly_fwd(s["x"], s["y"], s["plan"], s["desc"])
        B.bq_butterfly_bwd(s["x"], s["dy"], s["plan"], s["dx"], s["dtheta"], s["work"], s["desc"])
        return {"y": s["y"], "dx": s["dx"], "dtheta": s["dtheta"]}
    if op == "backward":
        B.bq_butterfly_bwd(s["x"], s["dy"], s["plan"], s["dx"], s["dtheta"], s["work"], s["desc"])
        return {"dx": s["dx"], "dtheta": s["dtheta"]}
    if op == "composite":
        (B.bq_kron_inv if s["inverse"] else B.bq_kron_fwd)(s["x"], s["y"], s["q1"], s["d1"], s["plan"], s["desc"])
        return s["y"]
    loss, grad, kl = s["cal"].loss_and_grad(s["x"])
    return {"loss": loss, "grad": grad, "kl": kl}


def work(case):
    """Bytes: every input read once, every output written once.  Flops: 3 n log2 n per application of a transform of
    n points (six per rotation), three applications and 4 flops per angle for the backward pass; dense products 2 per
    multiply-add."""
    op, n, rows, size = case["op"], case["n"], case["rows"], SIZE[case["dtype"]]
    k = n.bit_length() - 1
    if op == "calibrate":
        m = case["m"]
        angles = 4 * k * n // 2
        # two products for the error, two for its gradients; forward and backward transforms of both operands
        flops = 4 * 2.0 * rows * m * n + (rows + m) * (4 * 3.0 * n * k + 2.0 * n * k)
        return {"bytes": (rows + m) * n * size + 2 * angles, "flops": flops}
    if op == "composite":
        width = case["d1"] * n
        return {"bytes": 2 * rows * width * size, "flops": rows * (2.0 * case["d1"] * width + 3.0 * width * k)}
    width = n * case["heads"]
    row = width * size
    one = 3.0 * width * k
    angles = 4 * case["heads"] * k * n // 2
    coded = 0
    if "bits" in case:
        coded = width * case["bits"] // 8 + width // case["group"] * (2 if case["scale"] == "f16" else 4)
    if op == "quant":
        return {"bytes": rows * (row + coded) + angles, "flops": rows * one}
    if op == "transform":
        return {"bytes": 2 * rows * row + angles, "flops": rows * one}
    if op == "roundtrip":
        return {"bytes": rows * (3 * row + coded) + angles, "flops": rows * 3 * one}
    if op == "fakequant":
        return {"bytes": 2 * rows * row + angles, "flops": rows * one}
    back = 3 * one + 2.0 * width * k
    if op == "step":
        return {"bytes": 4 * rows * row + 2 * angles, "flops": rows * (one + back)}
    return {"bytes": 3 * rows * row + 2 * angles, "flops": rows * back}


def tolerance(case):
    """About four times what the path showed against the same arithmetic in 64 bits (or, for the calibration step, with
    its sums in 64 bits): the rounding of 16-bit outputs, the float32 cascade, and the codes and binary16 scales that a
    last-bit change of a rotated value moves across a rounding boundary."""
    op, dtype = case["op"], case["dtype"]
    if op == "calibrate":
        return {"rel": 1e-5, "max": 1e-4}
    if op == "quant":
        code_bytes = case["rows"] * case["n"] * case["heads"] * case["bits"] // 8
        return dict({"rel": 2e-4, "max": 4e-3} if case["scale"] == "f16" else {"rel": 5e-7, "max": 5e-6},
                    differ=min(0.01, 2e-5 + 2.0 / code_bytes))
    rows = {"f32": {"rel": 5e-7, "max": 2e-5}, "f16": {"rel": 8e-4, "max": 2e-3}, "bf16": {"rel": 7e-3, "max": 1.6e-2}}[dtype]
    if op == "composite":  # float32: sums of d1 products; 16-bit rows: some shapes round the butterfly's result as well
        return {"f32": {"rel": 2e-6, "max": 5e-5}, "f16": {"rel": 1.2e-3, "max": 3e-2}, "bf16": {"rel": 1e-2, "max": 0.2}}[dtype]
    if op == "roundtrip":
        code_bytes = case["rows"] * case["n"] * case["heads"] * case["bits"] // 8
        if case["scale"] == "f16":
            rows = {"rel": max(2e-4, rows["rel"]), "max": max(4e-3, rows["max"])}
        return dict(rows, differ=min(0.01, 2e-5 + 2.0 / code_bytes))
    if op == "fakequant":  # a code that moves by one moves its value by a whole quantisation step
        return {"rel": 2e-3, "max": 0.99}
    if op in ("step", "backward") and dtype == "f32":
        return {"rel": 1e-6, "max": 2e-5}
    return rows
