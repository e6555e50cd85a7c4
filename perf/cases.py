"""The work a program has this library do, as measured cases.

Kinds of work (one pass = what `run` does):
  fc        one quantized linear layer applied to a batch of activations (PackedLinear.__call__), bits_used chosen per call
  mlp       a forward pass of fully connected layers with bias and ReLU (pb_matmul_bias_act), one call per layer
  lstm      a sequence of LSTM cell steps on the fused gate matrix (pb_lstm_cell), hidden and cell state handed on
  shared    several weight matrices on the same activations (pb_act_prep once, then pb_matmul_prepared for each), on the
            layout of the AND + popcount kernel
  pack      Algorithm 1: fp32 weights to packed bitlayers and scales (pb_quantize_pack_mode)
  unpack    packed bitlayers back to integer codes (pb_unpack)

Everything is made on the GPU from the seed; weights are packed once in `prepare`, as a program does at load time.
"""
import math

import torch

from paper_2003_00822_amd import pb

LAYOUTS = {
    "bits": pb.PB_LAYOUT_TILE16_V1,          # the default
    "pairs": pb.PB_LAYOUT_TILE16_PAIRS_V1,   # for callers that serve batches
    "gates": pb.PB_LAYOUT_TILE16_GATES_V1,   # fused gate matrix of an LSTM
    "rows": pb.PB_LAYOUT_ROWMAJOR_V1,        # AND + popcount kernel
}
# position of the fixed point for the widths of the activations: N(0, 1) values keep a few integer bits
FRAC = {32: 16, 16: 12, 8: 4}


def listed():
    return [
        # The smallest layer of the benchmark's configurations: 1024 x 1024, 4 bits, one vector. Latency.
        {"name": "fc 1024 b4", "kind": "fc", "rows": 1024, "cols": 1024, "bits": 4, "used": 4, "batch": 1, "act_bits": 32,
         "layout": "bits"},
        # The headline layer, one vector, 3 of 8 stored bitlayers: the accuracy / speed knob in use.
        {"name": "fc 4096 b8 used3", "kind": "fc", "rows": 4096, "cols": 4096, "bits": 8, "used": 3, "batch": 1,
         "act_bits": 32, "layout": "bits"},
        # The largest layer of the benchmark, one vector, all bitlayers: the weight stream.
        {"name": "fc 16384 b8", "kind": "fc", "rows": 16384, "cols": 16384, "bits": 8, "used": 8, "batch": 1,
         "act_bits": 32, "layout": "bits"},
        # A handful of vectors on an odd-sized layer, odd bit counts, 16-bit activations (the paper's tables have 8, 16, 32).
        {"name": "fc ragged batch5 a16", "kind": "fc", "rows": 5003, "cols": 3001, "bits": 6, "used": 5, "batch": 5,
         "act_bits": 16, "layout": "bits"},
        # The large layer of the benchmark's batch configuration, default layout, 64 vectors.
        {"name": "fc 8192 b8 batch64", "kind": "fc", "rows": 8192, "cols": 8192, "bits": 8, "used": 8, "batch": 64,
         "act_bits": 32, "layout": "bits"},
        # The same layer served with the layout for batches, at the largest batch the benchmark runs.
        {"name": "fc 8192 b8 batch1024 pairs", "kind": "fc", "rows": 8192, "cols": 8192, "bits": 8, "used": 8,
         "batch": 1024, "act_bits": 32, "layout": "pairs"},
        # The 784-4096-4096-10 network, one input, 8-bit activations and 5 stored bitlayers as in the paper's model table.
        {"name": "mlp 784-4096-4096-10 a8", "kind": "mlp", "inputs": 784, "hidden": 4096, "outputs": 10, "bits": 5,
         "used": 5, "batch": 1, "act_bits": 8},
        # The LSTM of the benchmark's configurations: 35 dependent steps, one sequence; captured in a HIP graph, as the
        # library's sequences are meant to run.
        {"name": "lstm 1500 x35", "kind": "lstm", "hidden": 1500, "inputs": 1500, "steps": 35, "bits": 4, "used": 4,
         "batch": 1, "act_bits": 32, "layout": "gates", "graph": True},
        # Two matrices on one activation vector through the two-part calls, AND + popcount layout.
        {"name": "shared 4096 popcount", "kind": "shared", "rows": 4096, "rows2": 1000, "cols": 4096, "bits": 8, "used": 4,
         "batch": 1, "act_bits": 32, "layout": "rows"},
        # Quantize and pack the headline layer with the default quantizer.
        {"name": "pack 4096 b8", "kind": "pack", "rows": 4096, "cols": 4096, "bits": 8, "quantizer": "symmetric",
         "layout": "bits"},
        # Quantize an odd-sized layer with the clipping search, into the layout for batches.
        {"name": "pack ragged clip search", "kind": "pack", "rows": 3001, "cols": 5003, "bits": 4,
         "quantizer": "clip_search", "layout": "pairs"},
        # The codes of a large layer back as integers (checking, export).
        {"name": "unpack 8192 b8", "kind": "unpack", "rows": 8192, "cols": 8192, "bits": 8, "layout": "bits"},
    ]


def _spread(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]; every other one is odd."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choices(["fc", "mlp", "lstm", "shared", "pack", "unpack"], [8, 1, 2, 1, 3, 1])[0]
    bits = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 8, 12, 16])
    used = rng.randint(1, bits) if rng.random() < 0.5 else bits
    act_bits = rng.choice([32, 32, 16, 8])
    if kind == "fc":
        rows, cols = _spread(rng, 64, 16384), _spread(rng, 64, 16384)
        batch = 1 if rng.random() < 0.4 else _spread(rng, 1, 1024)
        while rows * cols * batch * bits > 8192 * 8192 * 1024 * 8:   # no more than the largest listed case
            batch = max(1, batch // 2)
        layout = "pairs" if batch > 8 and rng.random() < 0.5 else "bits"
        return {"kind": kind, "rows": rows, "cols": cols, "bits": bits, "used": used, "batch": batch, "act_bits": act_bits,
                "layout": layout}
    if kind == "mlp":
        return {"kind": kind, "inputs": _spread(rng, 100, 4096), "hidden": _spread(rng, 256, 8192),
                "outputs": _spread(rng, 2, 1000), "bits": bits, "used": used, "batch": rng.choice([1, 1, _spread(rng, 2, 64)]),
                "act_bits": act_bits}
    if kind == "lstm":
        hidden, inputs, steps = _spread(rng, 64, 3072), _spread(rng, 64, 3072), rng.randint(5, 35)
        batch = rng.choice([1, 1, _spread(rng, 2, 64)])
        while batch > 1 and 4 * hidden * (inputs + hidden) * steps * batch > 8192 * 8192 * 256:
            batch //= 2
        return {"kind": kind, "hidden": hidden, "inputs": inputs, "steps": steps, "bits": bits, "used": used, "batch": batch,
                "act_bits": act_bits, "layout": "gates", "graph": rng.random() < 0.5}
    if kind == "shared":
        return {"kind": kind, "rows": _spread(rng, 256, 8192), "rows2": _spread(rng, 256, 4096), "cols": _spread(rng, 256, 8192),
                "bits": min(bits, 8), "used": min(used, 8), "batch": rng.choice([1, 1, _spread(rng, 2, 16)]),
                "act_bits": act_bits, "layout": "rows"}
    rows, cols = _spread(rng, 64, 8192), _spread(rng, 64, 8192)
    layout = rng.choice(["bits", "bits", "pairs", "rows"])
    if kind == "pack":
        quantizer = rng.choice(["symmetric", "symmetric", "range", "sign", "clip_search"])
        while quantizer == "clip_search" and rows * cols > 1 << 24:   # (32 candidates per weight)
            rows //= 2
        return {"kind": kind, "rows": rows, "cols": cols, "bits": 2 if quantizer == "sign" else bits, "quantizer": quantizer,
                "layout": layout}
    return {"kind": kind, "rows": rows, "cols": cols, "bits": bits, "layout": layout}


def _desc(case, rows, cols):
    act = case.get("act_bits", 32)
    return pb.pb_desc_init_layout(rows, cols, case["bits"], LAYOUTS[case.get("layout", "bits")], frac_bits=FRAC[act],
                                  act_bits=act)


def _packed(case, rows, cols, normal, std):
    """A weight matrix ~N(0, std), packed: what a program keeps of it."""
    act = case.get("act_bits", 32)
    W = normal(rows, cols).mul_(std)
    return pb.PackedLinear(W, case["bits"], max_batch=case.get("batch", 1), frac_bits=FRAC[act], act_bits=act,
                           layout=LAYOUTS[case.get("layout", "bits")])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen)

    kind = case["kind"]
    s = {"case": case}
    if kind == "fc":
        s["lin"] = _packed(case, case["rows"], case["cols"], normal, 0.02)
        s["x"] = normal(case["batch"], case["cols"])
    elif kind == "mlp":
        dims = [case["inputs"], case["hidden"], case["hidden"], case["outputs"]]
        s["layers"] = [_packed(case, o, i, normal, 1.0 / math.sqrt(i)) for i, o in zip(dims, dims[1:])]
        s["bias"] = [normal(o).mul_(0.1) for o in dims[1:]]
        s["acts"] = [torch.empty((case["batch"], o), device="cuda") for o in dims[1:]]
        s["x"] = torch.rand((case["batch"], dims[0]), device="cuda", generator=gen)
    elif kind == "lstm":
        H, I, N = case["hidden"], case["inputs"], case["batch"]
        W = torch.rand((4 * H, I + H), device="cuda", generator=gen).sub_(0.5).mul_(0.08)
        act = case["act_bits"]
        s["lin"] = pb.PackedLinear(W, case["bits"], max_batch=N, frac_bits=FRAC[act], act_bits=act,
                                   layout=LAYOUTS[case["layout"]])
        s["bias"] = normal(4 * H).mul_(0.1)
        s["xs"] = [normal(N, I) for _ in range(case["steps"])]
        s["h"] = [torch.empty((N, H), device="cuda") for _ in range(case["steps"])]   # every step's hidden state
        s["c"] = torch.empty((N, H), device="cuda")
        s["zero"] = torch.zeros((N, H), device="cuda")
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _lstm_steps(s)   # once outside the capture
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                _lstm_steps(s)
    elif kind == "shared":
        s["lins"] = [_packed(case, r, case["cols"], normal, 0.02) for r in (case["rows"], case["rows2"])]
        s["x"] = normal(case["batch"], case["cols"])
        s["y"] = [torch.empty((case["batch"], r), device="cuda") for r in (case["rows"], case["rows2"])]
    elif kind == "pack":
        s["W"] = normal(case["rows"], case["cols"]).mul_(0.02)
        s["desc"] = _desc(case, case["rows"], case["cols"])
        s["packed"] = pb.alloc_packed(s["desc"])
        s["scales"] = torch.empty(case["bits"], device="cuda")
        s["quantizer"] = {"symmetric": pb.PB_QUANT_SYMMETRIC, "range": pb.PB_QUANT_RANGE, "sign": pb.PB_QUANT_SIGN,
                          "clip_search": pb.PB_QUANT_CLIP_SEARCH}[case["quantizer"]]
    elif kind == "unpack":
        lin = _packed(case, case["rows"], case["cols"], normal, 0.02)
        s["desc"], s["packed"] = lin.desc, lin.packed
        s["q"] = torch.empty((case["rows"], case["cols"]), dtype=torch.int32, device="cuda")
    return s


def _lstm_steps(s):
    case, lin = s["case"], s["lin"]
    h, c = s["zero"], s["zero"]
    for x, h_out in zip(s["xs"], s["h"]):
        pb.pb_lstm_cell(lin.packed, lin.scales, lin.desc, case["used"], x, case["inputs"], h, c, s["bias"], h_out, s["c"],
                        case["batch"], lin.workspace)
        h, c = h_out, s["c"]


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "fc":
        return s["lin"](s["x"], bits_used=case["used"])
    if kind == "mlp":
        x = s["x"]
        for i, lin in enumerate(s["layers"]):
            pb.pb_matmul_bias_act(lin.packed, lin.scales, lin.desc, case["used"], x, case["batch"], s["bias"][i],
                                  pb.PB_ACT_RELU if i < 2 else pb.PB_ACT_NONE, s["acts"][i], lin.workspace)
            x = s["acts"][i]
        return x
    if kind == "lstm":
        if case["graph"]:
            s["graph"].replay()
        else:
            _lstm_steps(s)
        return {"h": s["h"], "c": s["c"]}
    if kind == "shared":
        a, b = s["lins"]
        pb.pb_act_prep(a.desc, s["x"], case["batch"], a.workspace)
        for lin, y in ((a, s["y"][0]), (b, s["y"][1])):
            pb.pb_matmul_prepared(lin.packed, lin.scales, lin.desc, case["used"], case["batch"], y, a.workspace)
        return s["y"]
    if kind == "pack":
        pb.pb_quantize_pack_mode(s["W"], s["desc"], s["quantizer"], s["packed"], s["scales"])
        return {"packed": s["packed"], "scales": s["scales"]}
    pb.pb_unpack(s["packed"], s["desc"], s["q"])
    return s["q"]


def _product(rows, cols, used, batch):
    """Bytes and operations of one product: used bitlayers, activations and outputs once; a multiply-add per weight and vector."""
    return rows * cols * used / 8 + 4 * batch * (rows + cols), 2.0 * rows * cols * batch


def work(case):
    kind = case["kind"]
    if kind == "fc":
        parts = [_product(case["rows"], case["cols"], case["used"], case["batch"])]
    elif kind == "mlp":
        dims = [case["inputs"], case["hidden"], case["hidden"], case["outputs"]]
        parts = [_product(o, i, case["used"], case["batch"]) for i, o in zip(dims, dims[1:])]
    elif kind == "lstm":
        parts = [_product(4 * case["hidden"], case["inputs"] + case["hidden"], case["used"], case["batch"])] * case["steps"]
    elif kind == "shared":
        parts = [_product(r, case["cols"], case["used"], case["batch"]) for r in (case["rows"], case["rows2"])]
    else:
        n = case["rows"] * case["cols"]
        # 4 bytes of fp32 weight or int32 code and `bits` bits of packed code per element; about one operation each
        parts = [(n * (4 + case["bits"] / 8), n)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    kind = case["kind"]
    if kind == "pack":
        return {"rel": 1e-6, "max": 1e-6, "differ": 0.0}   # codes bit for bit; scales are fp32 products of one step
    if kind == "unpack":
        return "exact"
    if kind in ("mlp", "lstm") and case["act_bits"] < 32:
        # a value that falls on the other side of a step of the 8- or 16-bit grid between two layers moves by 2^-frac
        return {"rel": 2e-3}
    return {"rel": 1e-5}   # exact integer sums, scaled once, rounded once to fp32
