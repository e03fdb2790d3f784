"""The work that a training program has this library do, as a list of cases to time.

A case is one layer's share of a training step: the min-k drop of the layer's cached input
(``compress``) and the weight gradient from what was kept (``weight_grad``), called the way a
training program calls them -- inputs on the device, outputs and workspaces allocated once -- or,
for the ``layer`` cases, forward and backward of ``nn.Linear`` through autograd.  Shapes and value
distributions are those of the repository's benchmark workloads and of the DeiT-S-shaped encoder of
``block_bench`` (FC inputs after LayerNorm / GELU, convolution inputs after ReLU).
"""
import math

import torch

import paper_2202_13808_amd as dropit

# ---- the cases ------------------------------------------------------------------------------------
# kind   "fc": x [tokens, c_in] -> dW [c_out, c_in];  "conv": x [n, c, h, w] (layout nchw) or
#        [n, h, w, c] (nhwc), square window;  "layer": forward + backward of nn.Linear
# index  how the retained positions are kept: int32 flat indices, 16-bit in-row positions, bit mask


def _fc(name, dtype, tokens, c_in, c_out, gamma, dist, index="flat", kind="fc"):
    return {"name": name, "kind": kind, "dtype": dtype, "tokens": tokens, "c_in": c_in, "c_out": c_out,
            "gamma": gamma, "dist": dist, "index": index}


def _conv(name, dtype, n, c, h, w, c_out, kernel, stride, pad, gamma, layout, dist="relu"):
    return {"name": name, "kind": "conv", "dtype": dtype, "n": n, "c": c, "h": h, "w": w, "c_out": c_out,
            "kernel": kernel, "stride": stride, "pad": pad, "gamma": gamma, "dist": dist, "layout": layout}


def listed():
    return [
        # the smallest layer of the benchmark: launches and host time are all there is
        _fc("fc_tiny_f32", "f32", 256, 64, 128, 0.9, "normal"),
        # an encoder layer at a fine-tuning batch of 8 images of 197 tokens
        _fc("fc_batch8", "bf16", 8 * 197, 384, 1536, 0.9, "normal"),
        # ViT-B/16 MLP, first layer, batch 64: the benchmark's default workload
        _fc("fc_vitb_fc1", "bf16", 64 * 197, 768, 3072, 0.9, "normal"),
        # ViTDet-B MLP, second layer (GELU input): the largest tensor of the benchmark
        _fc("fc_vitdet_fc2", "bf16", 16384, 3072, 768, 0.9, "gelu"),
        # the same kind of layer in a program that trains in torch's default type
        _fc("fc_f32", "f32", 32 * 197, 384, 1536, 0.9, "normal"),
        # 16-bit in-row positions instead of int32 indices, at the rate where those start to pay
        _fc("fc_rows_form", "bf16", 128 * 197, 1536, 384, 0.8, "gelu", index="rows"),
        # forward and backward of one layer of the encoder through autograd, bit-mask form
        _fc("layer_mask_form", "bf16", 128 * 197, 384, 1152, 0.9, "normal", index="mask", kind="layer"),
        # ResNet-50 3x3 convolutions, early stage (large planes) and late stage (many channels)
        _conv("conv3x3_56", "bf16", 64, 64, 56, 56, 64, 3, 1, 1, 0.8, "nchw"),
        _conv("conv3x3_14", "bf16", 64, 256, 14, 14, 256, 3, 1, 1, 0.8, "nchw"),
        # the 1x1 convolution of a bottleneck
        _conv("conv1x1_56", "bf16", 64, 256, 56, 56, 64, 1, 1, 0, 0.8, "nchw"),
        # a program that trains in channels-last memory
        _conv("conv3x3_28_nhwc", "bf16", 64, 128, 28, 28, 128, 3, 1, 1, 0.8, "nhwc"),
        # ResNet-18 on 32x32 images in torch's default type
        _conv("conv3x3_f32", "f32", 32, 64, 32, 32, 64, 3, 1, 1, 0.8, "nchw"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A layer width: mostly a multiple of 8, sometimes any number."""
    v = _log_int(rng, lo, hi)
    return v if rng.random() < 0.2 else max(lo, v // 8 * 8)


def _draw_fc(rng):
    kind = rng.choice(["fc", "fc", "layer"])
    dtype = "bf16" if kind == "layer" else rng.choice(["bf16", "bf16", "bf16", "f32"])
    # (fp32 layers and odd output widths up to the size of the listed fp32 layer)
    c_out = _width(rng, 64, 3072)
    small = dtype == "f32" or c_out % 8 != 0
    tokens = _log_int(rng, 64, 8192 if small else 25216)
    return _fc("", dtype, tokens, _width(rng, 64, 3072), c_out, rng.choice([0.6, 0.7, 0.8, 0.9, 0.9]),
               rng.choice(["normal", "gelu"]), index=rng.choice(["flat", "flat", "rows", "mask"]), kind=kind)


def _draw_conv(rng):
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    layout = rng.choice(["nchw", "nchw", "nhwc"])
    kernel, stride, pad = rng.choice([(3, 1, 1), (3, 1, 1), (3, 1, 1), (1, 1, 0), (3, 2, 1), (1, 2, 0)])
    h = rng.randint(7, 64)
    w = h if rng.random() < 0.7 else rng.randint(7, 64)
    c = max(16, _log_int(rng, 16, 512) // 8 * 8)
    c_out = max(16, _log_int(rng, 16, 512) // 8 * 8)
    return _conv("", dtype, _log_int(rng, 2, 64), c, h, w, c_out, kernel, stride, pad, rng.choice([0.7, 0.8, 0.9]),
                 layout)


def draw(rng):
    limits = {c["name"]: work(c) for c in listed()}
    while True:
        case = _draw_fc(rng) if rng.random() < 0.55 else _draw_conv(rng)
        ceiling = limits["fc_vitdet_fc2"]
        if case["dtype"] == "f32":
            ceiling = limits["fc_f32" if case["kind"] == "fc" else "conv3x3_f32"]
        elif case["kind"] != "conv" and case["c_out"] % 8 != 0:
            ceiling = limits["fc_f32"]
        elif case["kind"] == "conv":
            ceiling = {"bytes": limits["conv1x1_56"]["bytes"], "flops": 4 * limits["conv3x3_56"]["flops"]}
        cost = work(case)
        if cost["bytes"] <= ceiling["bytes"] and cost["flops"] <= ceiling["flops"]:
            del case["name"]
            return case


# ---- shapes ---------------------------------------------------------------------------------------
def _shapes(case):
    """(x, dY, dW) shapes."""
    if case["kind"] != "conv":
        t, ci, co = case["tokens"], case["c_in"], case["c_out"]
        return (t, ci), (t, co), (co, ci)
    n, c, h, w, co, kn = (case[key] for key in ("n", "c", "h", "w", "c_out", "kernel"))
    oh, ow = ((e + 2 * case["pad"] - kn) // case["stride"] + 1 for e in (h, w))
    if case["layout"] == "nhwc":
        return (n, h, w, c), (n, oh, ow, co), (co, kn, kn, c)
    return (n, c, h, w), (n, co, oh, ow), (co, c, kn, kn)


def work(case):
    xs, ys, ws = _shapes(case)
    x, y, w = math.prod(xs), math.prod(ys), math.prod(ws)
    size = 2 if case["dtype"] == "bf16" else 4
    k = dropit.keep_count(x, case["gamma"])
    # the dense product over all positions of dY (the method keeps it dense): every output of the layer
    # is a sum over kernel * kernel * c_in inputs
    flops = 2 * y * (w // case["c_out"])
    # x and dY in; values, positions and dW out; values and positions are read again for the gradient
    index = {"flat": 4 * k, "rows": 2 * k + 4 * x // xs[-1], "mask": x // 8 + x // 256}[case.get("index", "flat")]
    moved = x * size + 2 * (k * size + index) + y * size + w * 4
    if case["kind"] == "layer":
        # y and dx out, weight in twice, dW in the weight's type; the three products of a linear layer
        return {"bytes": moved + x * size + y * size + 2 * w * size - w * (4 - size), "flops": 3 * flops}
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # Values, positions and offsets are the same bits whatever computes them.
    if case["kind"] == "layer":
        # y, dx, dW and db are rounded to bf16: 2^-9 of a value at most, 1.7e-3 in the 2-norm, on either side
        return {"rel": 5e-3}
    # fp32 sums: against the same sums in 64 bits the listed and ten drawn cases show 4e-8 to 4.5e-7 in the
    # 2-norm, and 5e-7 to 5e-6 of the root mean square in the worst element
    return {"rel": 2e-6, "max": 2e-5}


# ---- one pass -------------------------------------------------------------------------------------
_TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(seed)
    xs, ys, ws = _shapes(case)
    dtype = _TYPES[case["dtype"]]
    x = torch.randn(xs, generator=gen, device=dev)
    if case["dist"] == "relu":
        x = x.relu_()
    elif case["dist"] == "gelu":
        x = torch.nn.functional.gelu(x)
    x = x.to(dtype)
    dy = (torch.randn(ys, generator=gen, device=dev) * 0.02).to(dtype)
    state = {"case": case, "x": x, "dy": dy, "x_shape": xs}
    if case["kind"] == "layer":
        layer = dropit.nn.Linear(case["c_in"], case["c_out"], gamma=case["gamma"], index_format=case["index"],
                                 device=dev, dtype=dtype)
        with torch.no_grad():
            layer.weight.copy_(torch.randn(ws, generator=gen, device=dev) * case["c_in"] ** -0.5)
            layer.bias.copy_(torch.randn(ws[0], generator=gen, device=dev) * 0.02)
        state["layer"] = layer.train()
        state["x"] = x.requires_grad_(True)
        return state
    # what a training program keeps for the layer from step to step
    k = dropit.keep_count(x.numel(), case["gamma"])
    lib, code = dropit.lib(), dropit.binding._dtype_code(dtype)

    def space(size):
        return torch.empty(max(int(size), 256), dtype=torch.uint8, device=dev)

    index = case.get("index", "flat")
    state["conv"] = None
    if case["kind"] == "conv":
        kn, st, pd = case["kernel"], case["stride"], case["pad"]
        state["conv"] = (kn, kn, st, st, pd, pd, 1, 1)
    inner = dropit.weight_grad_workspace_bytes(xs, dtype, k, case["c_out"], state["conv"], layout=case.get("layout", "nchw"))
    state["dW"] = torch.empty(ws, dtype=torch.float32, device=dev)
    if index == "flat":
        state["vals"] = torch.empty(k, dtype=dtype, device=dev)
        state["idx"] = torch.empty(k, dtype=torch.int32, device=dev)
        state["ws_c"] = space(dropit.compress_workspace_bytes(x.numel(), dtype))
        state["ws_g"] = space(inner)
        return state
    shape = dropit.binding._shape_array(xs)
    if index == "rows":
        state["ws_c"] = space(lib.dropit_compress_rows_workspace_bytes(x.numel(), k, code))
        state["ws_g"] = space(lib.dropit_weight_grad_rows_workspace_bytes(shape, 2, code, k, case["c_out"], None))
    else:
        state["ws_c"] = space(lib.dropit_compress_mask_workspace_bytes(x.numel(), k, code))
        state["ws_g"] = space(lib.dropit_weight_grad_mask_workspace_bytes(shape, 2, code, k, case["c_out"], None))
    return state


def run(state):
    case = state["case"]
    x, dy = state["x"], state["dy"]
    if case["kind"] == "layer":
        layer = state["layer"]
        x.grad = layer.weight.grad = layer.bias.grad = None
        y = layer(x)
        y.backward(dy)
        return y.detach(), x.grad, layer.weight.grad, layer.bias.grad
    index = case.get("index", "flat")
    if index == "rows":
        vals, col, rowptr = dropit.compress_rows(x, case["gamma"], workspace=state["ws_c"])
        dw = dropit.weight_grad_rows(vals, col, rowptr, state["x_shape"], dy, case["c_out"], dW=state["dW"],
                                     workspace=state["ws_g"])
        return vals, col, rowptr, dw
    if index == "mask":
        vals, mask, blockptr = dropit.compress_mask(x, case["gamma"], workspace=state["ws_c"])
        dw = dropit.weight_grad_mask(vals, mask, blockptr, state["x_shape"], dy, case["c_out"], dW=state["dW"],
                                     workspace=state["ws_g"])
        return vals, mask, blockptr, dw
    vals, idx = dropit.compress(x, case["gamma"], vals=state["vals"], idx=state["idx"], workspace=state["ws_c"])
    dw = dropit.weight_grad(vals, idx, state["x_shape"], dy, case["c_out"], conv=state["conv"], dW=state["dW"],
                            workspace=state["ws_g"], layout=case.get("layout", "nchw"))
    return vals, idx, dw
