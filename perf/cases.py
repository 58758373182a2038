"""Performance cases: the sparse products and convolutions that users of this library run.

Every case is one inference call with a plan that was made beforehand: `sparsert.inspect` on the
pruned weights (once per layer, off the latency path), then `sparsert.spmm` / `sparsert.conv3x3` on
the activations of every call.  Weights are pruned to an exact nonzero count, as magnitude pruning
leaves them ("magnitude"), at random ("uniform"), or with rows of very different lengths
("skewed"); activations are N(0, 1), behind a ReLU for the 1x1 and 3x3 convolutions.

A case holds: op (spmm / conv), dtype (f32, f16 with fp32 sums, i8 with int32 results), the sizes
(M, K, N of C[M,N] = A[M,K] B[K,N]; Cout, Cin, img of a 3x3 / pad 1 convolution on img x img
pixels), batch (images or operand pairs per call), sparsity, mask, pad (elements by which the rows
of B and C lie further apart than N: a column slice of wider activations) and kernel ("auto": what
the inspector chooses, "rows": the executor whose plan needs no code generation).
"""
import math

import numpy as np
import torch

from paper_2008_11849_amd import sparsert as sp

_TORCH = {"f32": torch.float32, "f16": torch.float16, "i8": torch.int8}
_SIZE = {"f32": 4, "f16": 2, "i8": 1}
_OUT_TORCH = {"f32": torch.float32, "f16": torch.float16, "i8": torch.int32}
_OUT_SIZE = {"f32": 4, "f16": 2, "i8": 4}
_KERNEL = {"auto": sp.KERNEL_AUTO, "rows": sp.KERNEL_ROWS}

# Bounds of what draw() may give, taken from the largest listed cases.
_MAX_FLOPS = 2.7e9
_MAX_BYTES = 1.3e8
_MAX_NNZ_GENERATED = 260_000     # plan preparation (code generation) stays near a second
_MAX_NNZ_ROWS = 1_600_000


def _spmm(name, dtype, M, K, N, sparsity, mask="magnitude", batch=1, pad=0, kernel="auto", relu=False):
    return {"name": name, "op": "spmm", "dtype": dtype, "M": M, "K": K, "N": N, "sparsity": sparsity, "mask": mask,
            "batch": batch, "pad": pad, "kernel": kernel, "relu": relu}


def _conv(name, dtype, Cout, Cin, img, sparsity, batch=1, mask="magnitude", kernel="auto"):
    return {"name": name, "op": "conv", "dtype": dtype, "Cout": Cout, "Cin": Cin, "img": img, "sparsity": sparsity,
            "mask": mask, "batch": batch, "kernel": kernel, "relu": True}


def listed():
    return [
        # the smallest calls: a late MobileNet 1x1 convolution on one 7x7 image (ragged N); launch and latency bound
        _spmm("spmm_f32_1x1_7x7", "f32", 1024, 512, 49, 0.90, relu=True),
        # an ordinary 1x1 convolution, one 14x14 image (configuration c2)
        _spmm("spmm_f32_1x1_14x14", "f32", 512, 512, 196, 0.90, relu=True),
        # the two projections of a Transformer feed-forward layer, 8 x 128 tokens (configurations c3 and c3t)
        _spmm("spmm_f32_fc_up", "f32", 3072, 768, 1024, 0.95),
        _spmm("spmm_f32_fc_down", "f32", 768, 3072, 1024, 0.95),
        # the sparse end of the shape sweep at its largest size: many tokens through a wide layer
        _spmm("spmm_f32_large", "f32", 4096, 4096, 4096, 0.98, mask="uniform"),
        # rows of very different lengths (load balance), odd sizes, a column slice of wider activations
        _spmm("spmm_f32_skewed_slice", "f32", 1021, 1027, 771, 0.90, mask="skewed", pad=13),
        # a plan made without code generation (no assembler at hand, or no seconds to spend on it), many nonzeros
        _spmm("spmm_f32_rows_plan", "f32", 4096, 4096, 784, 0.90, mask="uniform", kernel="rows"),
        # the headline 3x3 convolution, one image (configuration c4)
        _conv("conv_f32_14x14", "f32", 256, 256, 14, 0.90),
        # a batch of eight images through an earlier 3x3 convolution, half storage
        _conv("conv_f16_28x28_b8", "f16", 128, 128, 28, 0.90, batch=8),
        # the up projection in half storage
        _spmm("spmm_f16_fc_up", "f16", 3072, 768, 1024, 0.95),
        # a moderately pruned square layer with many columns, half storage
        _spmm("spmm_f16_square", "f16", 1024, 1024, 4096, 0.80),
        # the down projection quantised to int8
        _spmm("spmm_i8_fc_down", "i8", 768, 3072, 1024, 0.95),
    ]


def _log_int(rng, lo, hi):
    """Log-uniform integer; two in three are rounded to a multiple of 8 or 64, as layer widths are."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    step = rng.choice([1, 8, 64])
    return int(min(hi, max(lo, round(v / step) * step)))


def draw(rng):
    """One more case: fp32 half of the time, one in four a convolution, sizes over the whole range."""
    while True:
        dtype = rng.choice(["f32", "f32", "f16", "i8"])
        mask = rng.choice(["magnitude", "magnitude", "uniform", "skewed"])
        kernel = rng.choice(["auto"] * 7 + ["rows"])
        sparsity = round(rng.uniform(0.80, 0.98), 3)
        if rng.random() < 0.25:
            case = _conv("", dtype, _log_int(rng, 32, 512), _log_int(rng, 32, 512), rng.randint(7, 56), sparsity,
                         batch=rng.choice([1, 1, 2, 8]), mask=mask, kernel=kernel)
        else:
            case = _spmm("", dtype, _log_int(rng, 64, 4096), _log_int(rng, 64, 4096), _log_int(rng, 49, 4096), sparsity,
                         mask=mask, batch=rng.choice([1, 1, 1, 4]), pad=rng.choice([0, 0, 0, rng.randint(1, 64)]),
                         kernel=kernel, relu=rng.random() < 0.3)
        del case["name"]
        w, nnz = work(case), _nnz(case)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES and nnz <= (_MAX_NNZ_ROWS if kernel == "rows" else _MAX_NNZ_GENERATED):
            return case


def _shape(case):
    if case["op"] == "conv":
        return case["Cout"], 9 * case["Cin"], case["img"] * case["img"]
    return case["M"], case["K"], case["N"]


def _nnz(case):
    M, K, _ = _shape(case)
    return max(1, round((1.0 - case["sparsity"]) * M * K))


def _weights(case, gen):
    """Pruned weights as host CSR (row_ptr, col_idx, vals), nonzero count fixed by the sparsity."""
    M, K, _ = _shape(case)
    w = torch.randn(M, K, generator=gen, device="cuda") * 0.02
    if case["mask"] == "skewed":   # Zipf-like row scales: after global pruning a few rows stay nearly dense
        w *= (1.0 + torch.randperm(M, generator=gen, device="cuda").to(torch.float32)).rsqrt()[:, None]
    score = torch.rand(M, K, generator=gen, device="cuda") if case["mask"] == "uniform" else w.abs()
    flat = torch.sort(score.reshape(-1), descending=True, stable=True).indices[:_nnz(case)]
    flat = torch.sort(flat).values
    vals = w.reshape(-1)[flat]
    vals = torch.where(vals == 0, torch.full_like(vals, 0.02), vals)
    if case["dtype"] == "i8":      # symmetric per tensor; a kept weight never becomes zero
        q = torch.round(vals / vals.abs().max() * 127.0)
        vals = torch.where(q == 0, torch.sign(vals), q)
    counts = torch.bincount(flat // K, minlength=M)
    row_ptr = np.zeros(M + 1, dtype=np.int32)
    row_ptr[1:] = torch.cumsum(counts, 0).to(torch.int32).cpu().numpy()
    return row_ptr, (flat % K).to(torch.int32).cpu().numpy(), vals.to(_TORCH[case["dtype"]]).cpu().numpy()


def _activations(case, gen, shape):
    x = torch.randn(*shape, generator=gen, device="cuda")
    if case["relu"]:
        x = torch.relu(x)
    if case["dtype"] == "i8":
        x = torch.clamp(torch.round(x * 32.0), -128, 127)
    return x.to(_TORCH[case["dtype"]])


def prepare(case, seed):
    """What an inference program holds before the call: the plan, the activations, the result buffer."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    M, K, N = _shape(case)
    batch, out = case["batch"], _OUT_TORCH[case["dtype"]]
    row_ptr, col_idx, vals = _weights(case, gen)
    stream = torch.cuda.current_stream().cuda_stream
    if case["op"] == "conv":
        img, Cin = case["img"], case["Cin"]
        plan = sp.inspect(row_ptr, col_idx, vals, M, K, N, conv=(Cin, img, img), batch=batch, kernel=_KERNEL[case["kernel"]])
        x = _activations(case, gen, (batch, Cin, img, img))
        y = torch.zeros(batch, M, img, img, dtype=out, device="cuda")
        return {"call": sp.conv3x3, "plan": plan, "x": x, "y": y, "stream": stream}
    ld = N + case["pad"]
    plan = sp.inspect(row_ptr, col_idx, vals, M, K, N, batch=batch, kernel=_KERNEL[case["kernel"]],
                      ldb=ld if case["pad"] else 0, ldc=ld if case["pad"] else 0)
    x = _activations(case, gen, (batch, K, ld))
    y = torch.zeros(batch, M, ld, dtype=out, device="cuda")
    return {"call": sp.spmm, "plan": plan, "x": x, "y": y, "stream": stream}


def run(state):
    """One inference call."""
    state["call"](state["plan"], state["x"].data_ptr(), state["y"].data_ptr(), state["stream"])
    return state["y"]


def work(case):
    """Activations and results once; of the weights the values and two bytes of position each, and the row pointer.
    Two operations per kept weight and column (convolution: per pixel at which the tap lies inside the image)."""
    M, K, N = _shape(case)
    nnz, e, o, batch = _nnz(case), _SIZE[case["dtype"]], _OUT_SIZE[case["dtype"]], case["batch"]
    if case["op"] == "conv":
        img = case["img"]
        inputs, columns = case["Cin"] * N, ((3 * img - 2) / 3.0) ** 2
    else:
        inputs, columns = K * N, N
    return {"bytes": batch * (e * inputs + o * M * N) + nnz * (e + 2) + 4 * (M + 1), "flops": 2.0 * nnz * columns * batch}


def tolerance(case):
    """fp32 sums in another order; one rounding to half of an fp32 sum; exact integers."""
    if case["dtype"] == "i8":
        return "exact"
    return {"rel": 1e-3, "max": 5e-3} if case["dtype"] == "f16" else {"rel": 1e-5, "max": 1e-4}
