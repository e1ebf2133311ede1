"""The work that programs have this library do, as cases that can be prepared, run and checked one by one.

Every case goes through the binding's public entry points, with what an inference program keeps between
calls (weights, offline weight checksums, plans, workspaces) made in ``prepare``.  The scheme is the library's
own choice (``AUTO``, or a plan's analytic selector) unless a case says otherwise, which is how the library is meant
to be used; the sticky fault flag comes back with every result.

Kinds of case and the ranges that ``draw`` covers:

* ``mlp``     DLRM's two MLPs (13-512-256-64 and 512-1024-1024-512-256-1, ReLU between the layers) as a plan, run
              with one call per pass; batch 1 .. 2048, fp16 / bf16.
* ``resnet``  ResNet-50's 53 convolutions at 224 x 224 as a plan, one call per pass; the three convolutions of a
              block are chained with ReLU, every block has an input of its own (pooling and the residual additions
              are no part of the library); batch 1 .. 4, fp16 / bf16.
* ``stem``    the first convolution of a CNN (7 x 7, stride 2, three input channels -> 64) as a plan; batch 1 .. 64,
              images of 160 .. 256 pixels, fp16 / bf16.
* ``block``   one bottleneck block (1 x 1 reduce, 3 x 3, 1 x 1 expand, ReLU after the first two) of one of the four
              stages as a plan; batch 4 .. 64, fp16 / bf16.
* ``gemm``    one linear layer called directly, with offline weight checksums: M 1 .. 8192, N and K 64 .. 8192
              (row-major weights and odd widths: M up to 2048, N and K up to 4096), fp16 / bf16 / int8.
* ``chain``   four equal layers handed to the library as a chain (ReLU between them), so that a layer can leave its
              successor's activation checksums; M 512 .. 4096, width 1024 .. 4096, fp16 / bf16.
"""
import math

import torch

from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

DEV = "cuda:0"
CODE = {"f16": B.F16, "bf16": B.BF16, "i8": B.I8}
TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8}
OUT = {"f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int32}


# ------------------------------------------------------------------------------------------------------------------ #
# the cases
# ------------------------------------------------------------------------------------------------------------------ #
def listed():
    return [
        # recommendation models at the smallest batch: eight launches, all latency
        {"name": "dlrm_batch1", "kind": "mlp", "dtype": "f16", "batch": 1},
        # the same at a serving batch
        {"name": "dlrm_batch256", "kind": "mlp", "dtype": "f16", "batch": 256},
        # image classification, one image: 53 small products, latency and too few tiles
        {"name": "resnet50_batch1", "kind": "resnet", "dtype": "f16", "batch": 1},
        # a CNN's first layer at a throughput batch: three channels, so no aligned chunks
        {"name": "stem_batch64", "kind": "stem", "dtype": "f16", "batch": 64, "size": 224},
        # the first stage's blocks at that batch: very many rows, 64 channels inside, memory traffic
        {"name": "block_stage1_batch64", "kind": "block", "dtype": "f16", "batch": 64, "stage": 1},
        # the third stage's blocks: 256 channels inside, mid-size products; bf16 as trained nowadays
        {"name": "block_stage3_batch64", "kind": "block", "dtype": "bf16", "batch": 64, "stage": 3},
        # a 4096-wide layer with sixteen rows (decoding a small batch): the weights' bytes
        {"name": "decode_16x4096x4096", "kind": "gemm", "dtype": "bf16", "M": 16, "N": 4096, "K": 4096, "layout": "nk", "dist": "weights"},
        # the same layer with 256 rows, just below the intensity where the scheme changes
        {"name": "layer_256x4096x4096", "kind": "gemm", "dtype": "f16", "M": 256, "N": 4096, "K": 4096, "layout": "nk", "dist": "weights"},
        # weights kept row-major (in x out) and sizes that fill no tile and no 16-byte chunk
        {"name": "odd_511x1000x2047_kn", "kind": "gemm", "dtype": "f16", "M": 511, "N": 1000, "K": 2047, "layout": "kn", "dist": "weights"},
        # quantised inference, compute bound
        {"name": "int8_4096", "kind": "gemm", "dtype": "i8", "M": 4096, "N": 4096, "K": 4096, "layout": "nk", "dist": "int8"},
        # prefill through four 4096-wide layers as a chain
        {"name": "chain4_2048x4096", "kind": "chain", "dtype": "bf16", "M": 2048, "width": 4096},
        # the largest product of the benchmark
        {"name": "square_8192", "kind": "gemm", "dtype": "f16", "M": 8192, "N": 8192, "K": 8192, "layout": "nk", "dist": "normal"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["mlp", "resnet", "stem", "block", "gemm", "gemm", "gemm", "gemm", "chain"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "mlp":
        return {"kind": kind, "dtype": dtype, "batch": _log_int(rng, 1, 2048)}
    if kind == "resnet":
        return {"kind": kind, "dtype": dtype, "batch": rng.randint(1, 4)}
    if kind == "stem":
        return {"kind": kind, "dtype": dtype, "batch": _log_int(rng, 1, 64), "size": rng.randint(160, 256)}
    if kind == "block":
        return {"kind": kind, "dtype": dtype, "batch": _log_int(rng, 4, 64), "stage": rng.randint(1, 4)}
    if kind == "chain":
        return {"kind": kind, "dtype": dtype, "M": _log_int(rng, 512, 4096), "width": 64 * rng.randint(16, 64)}
    dtype = rng.choice(["f16", "bf16", "i8"])
    layout = rng.choice(["nk", "nk", "nk", "kn"])
    odd = rng.random() < 0.3
    top = 8192 if layout == "nk" and not odd else 4096
    M, N, K = _log_int(rng, 1, top // 2 if top == 4096 else top), _log_int(rng, 64, top), _log_int(rng, 64, top)
    if not odd:  # most layers have widths of whole tiles; the rows are whatever the batch is
        N, K = -(-N // 64) * 64, -(-K // 128) * 128
    return {"kind": kind, "dtype": dtype, "M": M, "N": N, "K": K, "layout": layout,
            "dist": "int8" if dtype == "i8" else rng.choice(["weights", "normal"])}


# ------------------------------------------------------------------------------------------------------------------ #
# inputs, and what a program keeps
# ------------------------------------------------------------------------------------------------------------------ #
def _random(shape, dtype, dist, gen):
    if dtype == "i8":
        return torch.randint(-128, 128, shape, dtype=torch.int8, device=DEV, generator=gen)
    if dist == "uniform_01":
        x = torch.rand(shape, device=DEV, generator=gen)
    else:
        x = torch.randn(shape, device=DEV, generator=gen)
        if dist == "weights":
            x *= 0.02
    return x.to(TORCH[dtype])


class Plan:
    """A plan handle that lives as long as its state."""

    def __init__(self, layers):
        self.handle = B.abft_plan_create(layers)

    def __del__(self):
        if torch.cuda.is_available():
            torch.cuda.synchronize()
        B.abft_plan_destroy(self.handle)


def _network(case):
    """(layers, feeds, relu): the layers of a plan in order, for each the layer whose output it reads (None: an input of
    its own), and whether ReLU follows."""
    kind = case["kind"]
    if kind == "mlp":
        layers = wl.dlrm_layers(case["batch"])
        feeds = [None, 0, 1, None, 3, 4, 5, 6]
        relu = [True, True, False, True, True, True, True, False]
    elif kind == "resnet":
        layers = wl.resnet50_layers(case["batch"])
        feeds, relu = [], []
        for i, l in enumerate(layers):
            inner = l.name.endswith((".conv2", ".conv3"))
            feeds.append(i - 1 if inner else None)
            relu.append(not l.name.endswith((".conv3", ".downsample")))
    elif kind == "stem":
        layers = wl.resnet50_layers(case["batch"], case["size"], case["size"])[:1]
        feeds, relu = [None], [True]
    elif kind == "block":
        name = f"layer{case['stage']}.1."
        layers = [l for l in wl.resnet50_layers(case["batch"]) if l.name.startswith(name)]
        feeds, relu = [None, 0, 1], [True, True, False]
    else:
        w = case["width"]
        layers = [wl.Layer(f"chain{i}", case["M"], w, w) for i in range(4)]
        feeds, relu = [None, 0, 1, 2], [True, True, True, False]
    return layers, feeds, relu


def _inputs(case, gen):
    """Inputs and weights (N x K) of a network case, in a fixed order."""
    layers, feeds, relu = _network(case)
    xs, ws = [], []
    for l, f in zip(layers, feeds):
        c = l.conv
        shape = (l.M, l.K) if c is None else (c.batch, c.H, c.W, c.Cin)
        xs.append(None if f is not None else _random(shape, case["dtype"], "uniform_01", gen))
        ws.append(_random((l.N, l.K), case["dtype"], "weights", gen))
    return layers, feeds, relu, xs, ws


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _product(case, gen):
    dist_a = "int8" if case["dtype"] == "i8" else "normal"
    A = _random((case["M"], case["K"]), case["dtype"], dist_a, gen)
    shape = (case["N"], case["K"]) if case["layout"] == "nk" else (case["K"], case["N"])
    return A, _random(shape, case["dtype"], case["dist"], gen)


def prepare(case, seed):
    gen = _generator(seed)
    dt = CODE[case["dtype"]]
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    if case["kind"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        A, W = _product(case, gen)
        layout = B.B_NK if case["layout"] == "nk" else B.B_KN
        aligned = layout == B.B_NK and K * A.element_size() % 16 == 0
        _, block_n = B.abft_region_shape(M, N, K, dt, aligned)
        beta = torch.zeros(B.abft_beta_bytes(K, N, block_n), dtype=torch.uint8, device=DEV)
        B.abft_weight_checksum(K, N, W, W.shape[1], layout, dt, beta, block_n=block_n)
        nws = B.abft_workspace_bytes(M, N, K, dt, B.AUTO)
        ws = torch.empty(nws, dtype=torch.uint8, device=DEV) if nws else None
        C = torch.zeros((M, N), dtype=OUT[case["dtype"]], device=DEV)
        return {"kind": "gemm", "dims": (M, N, K), "A": A, "W": W, "layout": layout, "C": C, "dtype": dt, "beta": beta,
                "ws": ws, "nws": nws, "flag": flag}
    layers, feeds, relu, xs, ws = _inputs(case, gen)
    outs = [torch.zeros((l.M, l.N), dtype=OUT[case["dtype"]], device=DEV) for l in layers]
    descs = []
    for l, w in zip(layers, ws):
        c = l.conv
        geo = B.Conv(c.batch, c.H, c.W, c.Cin, c.KH, c.KW, c.stride, c.pad) if c is not None else B.Conv()
        descs.append(B.Layer(l.M, l.N, l.K, dt, B.B_NK, 0 if c is None else 1, geo, w.data_ptr(), l.K))
    plan = Plan(descs)
    for i, r in enumerate(relu):
        if r:
            B.abft_plan_set_activation(plan.handle, i, B.ACT_RELU)
    state = {"kind": case["kind"], "plan": plan, "weights": ws, "inputs": xs, "outs": outs, "flag": flag}
    if case["kind"] == "chain":
        state["width"] = case["width"]
    else:
        ins = [x if f is None else outs[f] for x, f in zip(xs, feeds)]
        state["io"] = B.PlanIO(ins, [l.K for l in layers], outs, [l.N for l in layers])
    return state


def run(state):
    if state["kind"] == "gemm":
        (M, N, K), W = state["dims"], state["W"]
        B.abft_gemm(M, N, K, state["A"], K, W, W.shape[1], state["layout"], state["C"], N, state["dtype"], B.AUTO,
                    beta=state["beta"], workspace=state["ws"], workspace_bytes=state["nws"], fault_flag=state["flag"])
        return state["C"], state["flag"]
    if state["kind"] == "chain":
        w = state["width"]
        B.abft_plan_run_chain(state["plan"].handle, 0, 4, state["inputs"][0], w, state["outs"], [w] * 4, state["flag"])
    else:
        B.abft_plan_run_all(state["plan"].handle, state["io"], state["flag"])
    return state["outs"], state["flag"]


# ------------------------------------------------------------------------------------------------------------------ #
# what a pass cannot do without, and what it has to give
# ------------------------------------------------------------------------------------------------------------------ #
def work(case):
    es, cs = (1, 4) if case["dtype"] == "i8" else (2, 2)
    if case["kind"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": es * (M * K + N * K) + cs * M * N, "flops": 2 * M * N * K}
    layers, feeds, _ = _network(case)
    total = flops = 0
    for l, f in zip(layers, feeds):
        c = l.conv
        # a layer's input counts where it comes from outside; what an earlier layer left is counted there, as its output
        x = 0 if f is not None else (l.M * l.K if c is None else c.batch * c.H * c.W * c.Cin)
        total += es * (x + l.N * l.K) + cs * l.M * l.N
        flops += 2 * l.M * l.N * l.K
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """int8 is exact.  fp16 / bf16: results are rounded once to their type, so against another order of the fp32 sums
    some fall to the neighbouring value, and networks carry such a change through the layers that follow.  `rel` is
    four times the distance from the 64-bit result that is seen: fp16 2.1e-4 for one product, 3.7e-4 behind the
    convolutions of a block, 1e-3 at the single output that ends DLRM's five layers; bf16 eight times that (its unit
    roundoff), which for one product is 1.7e-3 and behind four chained layers 3.3e-3.  `max`: some ulps."""
    if case["dtype"] == "i8":
        return "exact"
    rel = {"gemm": 8.5e-4, "mlp": 4e-3}.get(case["kind"], 1.6e-3)
    if case["dtype"] == "f16":
        return {"rel": rel, "max": 10 * rel}
    return {"rel": min(8 * rel, 0.03), "max": min(80 * rel, 0.3)}


def _columns(x, c):
    """The lowered activations of a convolution: (batch * OH * OW) x (KH * KW * Cin)."""
    if c.KH == 1 and c.KW == 1 and c.pad == 0:
        return x[:, :: c.stride, :: c.stride, :].reshape(-1, c.Cin)
    p = c.pad
    xp = torch.zeros((x.shape[0], c.H + 2 * p, c.W + 2 * p, c.Cin), dtype=x.dtype, device=x.device)
    xp[:, p:p + c.H, p:p + c.W, :] = x
    taps = [xp[:, kh:kh + (c.OH - 1) * c.stride + 1:c.stride, kw:kw + (c.OW - 1) * c.stride + 1:c.stride, :]
            for kh in range(c.KH) for kw in range(c.KW)]
    return torch.cat(taps, dim=-1).reshape(-1, c.KH * c.KW * c.Cin)


def exact(case, seed):
    gen = _generator(seed)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    if case["kind"] == "gemm":
        if case["dtype"] == "i8":
            return None
        A, W = _product(case, gen)
        W = W.double()
        return A.double() @ (W.t() if case["layout"] == "nk" else W), flag
    layers, feeds, relu, xs, ws = _inputs(case, gen)
    outs = []
    for l, f, r, x, w in zip(layers, feeds, relu, xs, ws):
        x = outs[f] if f is not None else x.double()
        c = l.conv
        if c is None:
            y = x @ w.double().t()
        else:
            step = max(1, 16 * 1024 * 1024 // (c.OH * c.OW * l.K))  # images at a time, for the lowered copy's size
            x = x.reshape(c.batch, c.H, c.W, c.Cin)
            y = torch.cat([_columns(x[i:i + step], c) @ w.double().t() for i in range(0, c.batch, step)])
        outs.append(torch.relu(y) if r else y)
    return outs, flag
