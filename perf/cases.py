"""What this library is timed on: whole networks, blocks, modules, single layers and the fitting step of a slim layer,
through the entry points of ``paper_1708_04728_amd.binding``, from one image to a batch of 128.

A case names a path ("net", "module", "conv", "fit"), the structure it runs, its form, its sizes and how it is launched:

* form "original": every layer a kernel of its own (the form the slim one is compared with); "fused": the original
  structure with ReLU, concat and the stacked first steps in the convolutions' stores and max-pool + LRN in one pass
  (how a network that has not been slimmed is deployed); "slim": the slimmed structure with the same fusions.
* fp32 runs on NCHW tensors, bf16 on channels-last ones; filters are packed once where their channel count allows it.
* launch "graph": the forward recorded once and launched as one HIP graph, branches of the four-branch modules side by
  side; "eager": call by call.

Inputs and weights are drawn on the device from the seed: images N(0,1), feature maps after a ReLU |N(0,1)| or U[0,1),
filters He-normal, biases N(0, 0.01^2), BatchNorm statistics U[0.5,1.5) / N(0, 0.1^2).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1708_04728_amd import binding as B, graph as G, slim as S

BN_EPS = 1e-5
LRN5 = {"n": 5, "alpha": 1e-4, "beta": 0.75, "k": 1.0}
FUSE = B.DR_FUSE_RELU | B.DR_FUSE_CONCAT | B.DR_FUSE_STACK

# GoogLeNet's inception modules: in, 1x1, 3x3 reduce, 3x3, 5x5 reduce, 5x5, pool projection; side of the module's map
MODULES = {
    "3a": (192, 64, 96, 128, 16, 32, 32, 28), "3b": (256, 128, 128, 192, 32, 96, 64, 28),
    "4a": (480, 192, 96, 208, 16, 48, 64, 14), "4b": (512, 160, 112, 224, 24, 64, 64, 14),
    "4c": (512, 128, 128, 256, 24, 64, 64, 14), "4d": (512, 112, 144, 288, 32, 64, 64, 14),
    "4e": (528, 256, 160, 320, 32, 128, 128, 14),
    "5a": (832, 256, 160, 320, 32, 128, 128, 7), "5b": (832, 384, 192, 384, 48, 128, 128, 7),
}


def listed():
    return [
        # -- the smallest calls: one image, where launches and latency count (the setting of the paper's own timings)
        # GoogLeNet's second block, slimmed: one strided convolution on one image
        dict(name="streamline_slim_f32_b1", path="net", net="streamline", form="slim", dtype="f32", batch=1, c=64, k=192, h=56, w=56, launch="eager"),
        # the same block as it was: convolution, ReLU, LRN, max-pool
        dict(name="streamline_original_f32_b1", path="net", net="streamline", form="original", dtype="f32", batch=1, c=64, k=192, h=56, w=56, launch="eager"),
        # classification of one image by the slim network, call by call
        dict(name="googlenet_slim_bf16_b1", path="net", net="googlenet", form="slim", dtype="bf16", batch=1, launch="eager"),
        # -- ordinary calls
        # one inception module in fp32 as a block benchmark runs it, slimmed
        dict(name="inception3a_slim_f32_b32", path="module", module="3a", form="slim", dtype="f32", batch=32, h=28, w=28),
        # a module of a network that runs on another image size, odd batch and ragged map
        dict(name="inception4c_fused_bf16_b37", path="module", module="4c", form="fused", dtype="bf16", batch=37, h=15, w=13),
        # a serving batch of the network that has not been slimmed
        dict(name="googlenet_fused_bf16_b19", path="net", net="googlenet", form="fused", dtype="bf16", batch=19, launch="eager"),
        # one layer with a channel count that fits no tile, on a wide odd map
        dict(name="conv5x5_bf16_ragged", path="conv", dtype="bf16", batch=9, c=24, k=88, r=5, stride=1, h=31, w=45),
        # learning a slim layer: forward, loss, parameter gradients, descent step
        dict(name="fit_slim_layer_f32_b32", path="fit", dtype="f32", batch=32, c=64, k=192, h=56, w=56),
        # -- the largest: throughput of a full batch
        dict(name="alexnet_front_original_f32_b128", path="net", net="alexnet_front", form="original", dtype="f32", batch=128, launch="eager"),
        dict(name="resnet_conv2x_slim_bf16_b128", path="net", net="resnet_conv2_x", form="slim", dtype="bf16", batch=128, h=56, w=56, launch="eager"),
        dict(name="googlenet_slim_bf16_b128", path="net", net="googlenet", form="slim", dtype="bf16", batch=128, launch="graph"),
        dict(name="googlenet_original_bf16_b128", path="net", net="googlenet", form="original", dtype="bf16", batch=128, launch="graph"),
    ]


def _log(rng, lo, hi):
    """A whole number whose logarithm is spread evenly over [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("googlenet", "googlenet", "googlenet", "module", "module", "conv", "conv", "streamline", "alexnet_front", "resnet_conv2_x", "fit"))
    if kind == "googlenet":
        return dict(path="net", net=kind, form=rng.choice(("original", "fused", "slim", "slim")), dtype="bf16", batch=_log(rng, 1, 128),
                    launch=rng.choice(("eager", "graph")))
    if kind == "alexnet_front":
        return dict(path="net", net=kind, form=rng.choice(("original", "fused", "slim")), dtype="f32", batch=_log(rng, 1, 128), launch=rng.choice(("eager", "graph")))
    if kind == "resnet_conv2_x":
        return dict(path="net", net=kind, form=rng.choice(("original", "slim")), dtype="bf16", batch=_log(rng, 1, 128), h=rng.randint(28, 56), w=rng.randint(28, 56),
                    launch=rng.choice(("eager", "graph")))
    if kind == "streamline":
        return dict(path="net", net=kind, form=rng.choice(("original", "fused", "slim")), dtype="f32", batch=_log(rng, 1, 32), c=rng.choice((32, 64, 96)),
                    k=rng.choice((96, 128, 192, 256)), h=_log(rng, 14, 56), w=_log(rng, 14, 56), launch="eager")
    if kind == "module":
        m, dtype = rng.choice(sorted(MODULES)), rng.choice(("f32", "bf16", "bf16"))
        side = MODULES[m][7]
        return dict(path="module", module=m, form=rng.choice(("original", "fused", "slim")), dtype=dtype, batch=_log(rng, 1, 64 if dtype == "f32" else 128),
                    h=rng.randint(side - side // 4, side + side // 4), w=rng.randint(side - side // 4, side + side // 4))
    if kind == "fit":
        return dict(path="fit", dtype="f32", batch=_log(rng, 1, 32), c=rng.choice((32, 64)), k=rng.choice((64, 96, 128, 192)), h=2 * _log(rng, 7, 28), w=2 * _log(rng, 7, 28))
    dtype = rng.choice(("f32", "bf16", "bf16"))
    q = dict(path="conv", dtype=dtype, batch=_log(rng, 1, 64), c=8 * _log(rng, 2, 64) if dtype == "bf16" else 16 * _log(rng, 1, 16), k=8 * _log(rng, 2, 48), r=rng.choice((1, 3, 3, 5)),
             stride=rng.choice((1, 1, 1, 2)), h=_log(rng, 7, 112), w=_log(rng, 7, 112))
    while work(q)["flops"] > (8e10 if dtype == "bf16" else 2e10) or work(q)["bytes"] > 6e8:
        q["batch"], q["h"] = max(1, q["batch"] // 2), q["h"] if q["batch"] > 1 else max(7, q["h"] // 2)
    return q


# ---- structures ------------------------------------------------------------------------------------------------------
def _conv(k, r, stride=1, pad=0):
    return ("conv", {"k": k, "r": r, "s": r, "stride": stride, "pad": pad})


_RELU, _LRN = ("relu", {}), ("lrn", LRN5)


def _pool(k, stride, pad=0):
    return ("maxpool", {"k": k, "stride": stride, "pad": pad})


def _inception(m):
    _, c1, c3r, c3, c5r, c5, cp, _ = MODULES[m]
    return ("inception", {"branches": [[_conv(c1, 1), _RELU], [_conv(c3r, 1), _RELU, _conv(c3, 3, 1, 1), _RELU], [_conv(c5r, 1), _RELU, _conv(c5, 5, 1, 2), _RELU],
                                       [_pool(3, 1, 1), _conv(cp, 1), _RELU]]})


def _structure(case):
    """(layer list of the case's form, shape of one input image (c, h, w))"""
    if case["path"] == "module":
        layers, shape = [_inception(case["module"])], (MODULES[case["module"]][0], case["h"], case["w"])
    elif case["net"] == "streamline":
        layers, shape = [_conv(case["k"], 3, 1, 1), _RELU, _LRN, _pool(3, 2)], (case["c"], case["h"], case["w"])
    elif case["net"] == "alexnet_front":
        layers, shape = [_conv(96, 11, 4), _RELU, _LRN, _pool(3, 2), _conv(256, 5, 1, 2), _RELU, _LRN, _pool(3, 2)], (3, 227, 227)
    elif case["net"] == "resnet_conv2_x":
        return [("bottleneck", {"mid": 64, "out": 256, "project": i == 0, "eps": BN_EPS}) for i in range(3)], (64, case["h"], case["w"])
    else:
        inc = [_inception(m) for m in sorted(MODULES)]
        layers = ([_conv(64, 7, 2, 3), _RELU, _pool(3, 2), _LRN, _conv(64, 1), _RELU, _conv(192, 3, 1, 1), _RELU, _LRN, _pool(3, 2)] + inc[:2] + [_pool(3, 2)] + inc[2:7]
                  + [_pool(3, 2)] + inc[7:] + [("avgpool", {"k": 7}), ("fc", {"out": 1000}), ("softmax", {})])
        shape = (3, 224, 224)
    return (S.slim_network(layers) if case["form"] == "slim" else layers), shape


# ---- inputs and parameters ---------------------------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _input(case, gen, shape, values):
    """An input tensor in the order its data type runs in: bf16 channels-last, fp32 NCHW."""
    n, (c, h, w) = case["batch"], shape
    bf16 = case["dtype"] == "bf16"
    dims = (n, h, w, c) if bf16 else (n, c, h, w)
    t = torch.rand(dims, device="cuda", generator=gen) if values == "uniform" else torch.randn(dims, device="cuda", generator=gen)
    t = (t.abs() if values == "absnormal" else t).to(_dtype(case))
    return B.NHWC(t) if bf16 else t


def _weights(case, gen, k, c, r, pack=True):
    w = (torch.randn((k, c, r, r), device="cuda", generator=gen) * math.sqrt(2.0 / (c * r * r))).to(_dtype(case))
    return (B.pack_filters(w) if pack and B.can_pack(c, case["dtype"]) else w), torch.randn(k, device="cuda", generator=gen) * 0.01


def _params(case, gen, layers, c, out):
    """Appends the parameters of a layer list in forward order; returns the channels it ends with."""
    for kind, p in layers:
        if kind == "conv":
            out += _weights(case, gen, p["k"], c, p["r"])
            c = p["k"]
        elif kind == "inception":
            c = sum(_params(case, gen, br, c, out) for br in p["branches"])
        elif kind == "bottleneck":
            for k, r, ci in ((p["mid"], 1, c), (p["mid"], 3, p["mid"]), (p["out"], 1, p["mid"])) + (((p["out"], 1, c),) if p["project"] else ()):
                bn = [torch.rand(k, device="cuda", generator=gen) + 0.5, torch.randn(k, device="cuda", generator=gen) * 0.1,
                      torch.randn(k, device="cuda", generator=gen) * 0.1, torch.rand(k, device="cuda", generator=gen) + 0.5]
                if case["form"] == "slim":      # BatchNorm folded into the filters, once, by the library's host routine
                    w, b = _weights(dict(case, dtype="f32"), gen, k, ci, r, pack=False)
                    wf, bf = B.fold_bn(w.cpu().numpy(), b.cpu().numpy(), *[v.cpu().numpy() for v in bn], float(np.float32(BN_EPS)))
                    out += [B.pack_filters(torch.from_numpy(wf).cuda().to(_dtype(case))), torch.from_numpy(bf).cuda()]
                else:
                    out += [*_weights(case, gen, k, ci, r), *bn]
            c = p["out"]
        elif kind == "fc":
            # Xavier, as classifiers are initialised: logits of a few units, so that the probabilities are not one-hot
            out += [(torch.randn((p["out"], c), device="cuda", generator=gen) * math.sqrt(1.0 / c)).to(_dtype(case)), torch.randn(p["out"], device="cuda", generator=gen) * 0.01]
            c = p["out"]
    return c


def _scratch(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return {"net": _prepare_net, "module": _prepare_module, "conv": _prepare_conv, "fit": _prepare_fit}[case["path"]](case, gen)


def _prepare_net(case, gen):
    layers, shape = _structure(case)
    values = {"streamline": "uniform", "resnet_conv2_x": "absnormal"}.get(case["net"], "normal")
    x = _input(case, gen, shape, values)
    params = []
    _params(case, gen, layers, shape[0], params)
    plain = case["form"] == "original"
    four = case["form"] != "slim" and case["launch"] == "graph"       # four branches side by side pay inside a graph
    net = B.Net(G.net_descs(layers, shape[0], inception_mode=(0 if plain else FUSE) | (B.DR_CONCURRENT_BRANCHES if four else 0), fuse_relu=not plain,
                            folded=case["form"] == "slim", pack=case["dtype"], fuse_nontensor=case["form"] == "fused" and case["dtype"] == "bf16"))
    if not plain and case["net"] == "googlenet":
        params = G.stack_first_steps(layers, params)
    xd = B.desc(x)
    y, ws = G.empty_like_desc(net.output_desc(xd)), _scratch(net.workspace_bytes(xd))
    state = dict(call=_run_net, net=net, x=x, params=params, y=y, ws=ws, graph=None)
    if case["launch"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        state["graph"] = net.capture(x, params, y, ws, side)
    return state


def _run_net(s):
    if s["graph"] is not None:
        s["graph"].launch()
    else:
        s["net"].fwd(s["x"], s["params"], s["y"], s["ws"])
    return s["y"].t if isinstance(s["y"], B.NHWC) else s["y"]


def _prepare_module(case, gen):
    layers, shape = _structure(case)
    x = _input(case, gen, shape, "absnormal")
    params = []
    c_out = _params(case, gen, layers, shape[0], params)
    if case["form"] != "original":
        params = G.stack_first_steps(layers, params)
    desc = G.inception_desc(layers[0][1], shape[0], 0 if case["form"] == "original" else FUSE, case["dtype"])
    dims = (case["batch"], case["h"], case["w"], c_out) if case["dtype"] == "bf16" else (case["batch"], c_out, case["h"], case["w"])
    y = torch.empty(dims, dtype=_dtype(case), device="cuda")
    return dict(call=_run_module, x=x, desc=desc, weights=params[0::2], biases=params[1::2], y=B.NHWC(y) if case["dtype"] == "bf16" else y,
                out=y, ws=_scratch(B.inception_workspace_bytes(x, desc)))


def _run_module(s):
    B.inception_fwd(s["x"], s["desc"], s["weights"], s["biases"], s["y"], s["ws"])
    return s["out"]


def _conv_out(case):
    pad = case["r"] // 2
    return tuple((case[d] + 2 * pad - case["r"]) // case["stride"] + 1 for d in ("h", "w"))


def _prepare_conv(case, gen):
    x = _input(case, gen, (case["c"], case["h"], case["w"]), "absnormal")
    w, b = _weights(case, gen, case["k"], case["c"], case["r"])
    cd = G.conv_desc(dict(k=case["k"], r=case["r"], s=case["r"], stride=case["stride"], pad=case["r"] // 2), case["c"], relu=True, pack=case["dtype"])
    p, q = _conv_out(case)
    y = torch.empty((case["batch"], p, q, case["k"]) if case["dtype"] == "bf16" else (case["batch"], case["k"], p, q), dtype=_dtype(case), device="cuda")
    need = B.conv2d_workspace_bytes(x, cd)
    return dict(call=_run_conv, x=x, cd=cd, w=w, b=b, y=B.NHWC(y) if case["dtype"] == "bf16" else y, out=y, ws=_scratch(need) if need else None)


def _run_conv(s):
    B.conv2d_fwd_ws(s["x"], s["cd"], s["w"], s["b"], s["y"], s["ws"])
    return s["out"]


def _prepare_fit(case, gen):
    # the target is the feature map of the block that the slim layer replaces
    block = _prepare_net(dict(case, path="net", net="streamline", form="original", launch="eager"), gen)
    _run_net(block)
    x, y = block["x"], block["y"]
    w, b = _weights(case, gen, case["k"], case["c"], 3, pack=False)
    slim = B.conv_desc(case["k"], case["c"], 3, 3, 2, 1, True, B.DR_KCRS)
    f = torch.empty_like(y)
    pixels = f.shape[0] * f.shape[2] * f.shape[3]
    return dict(call=_run_fit, x=x, y=y, f=f, w=w, b=b, dw=torch.empty_like(w), db=torch.empty_like(b), loss=torch.zeros(1, device="cuda"), slim=slim,
                conv=B.conv_desc(case["k"], case["c"], 3, 3, 1, 1, False, B.DR_KCRS),
                # below 2 / (largest curvature of the loss), which grows with the number of pixels and of weights per filter
                lr=2.9 / (pixels * case["c"] * 9), ws=_scratch(max(B.conv2d_bwd_params_workspace_bytes(x, slim), B.regression_loss_workspace_bytes())))


def _run_fit(s):
    B.slim_conv_fwd(s["x"], s["conv"], 2, s["w"], s["b"], s["f"])
    B.regression_loss_grad(s["f"], s["y"], s["f"], s["loss"], s["ws"])
    B.conv2d_bwd_params(s["x"], s["slim"], s["f"], s["dw"], s["db"], s["ws"])
    B.sgd_step(s["w"], s["dw"], s["lr"])
    B.sgd_step(s["b"], s["db"], s["lr"])
    return {"loss": s["loss"], "dw": s["dw"], "db": s["db"], "w": s["w"], "b": s["b"]}


def run(state):
    return state["call"](state)


# ---- what a pass cannot do without ---------------------------------------------------------------------------------------
def _walk(layers, shape, tot):
    """Adds the FLOP and the parameter elements of one image's forward to tot; returns the output's shape."""
    c, h, w = shape

    def conv(k, r, ci, p, q):
        tot["flops"] += 2.0 * k * ci * r * r * p * q
        tot["weights"] += k * ci * r * r

    for kind, p in layers:
        if kind == "conv":
            h, w = ((d + 2 * p["pad"] - p["r"]) // p["stride"] + 1 for d in (h, w))
            conv(p["k"], p["r"], c, h, w)
            c = p["k"]
        elif kind == "maxpool":
            h, w = (-(-(d + 2 * p["pad"] - p["k"]) // p["stride"]) + 1 for d in (h, w))
        elif kind == "inception":
            c = sum(_walk(br, (c, h, w), tot)[0] for br in p["branches"])
        elif kind == "bottleneck":
            for k, r, ci in ((p["mid"], 1, c), (p["mid"], 3, p["mid"]), (p["out"], 1, p["mid"])) + (((p["out"], 1, c),) if p["project"] else ()):
                conv(k, r, ci, h, w)
            c = p["out"]
        elif kind == "avgpool":
            h, w = h - p["k"] + 1, w - p["k"] + 1
        elif kind == "fc":
            conv(p["out"], 1, c * h * w, 1, 1)
            c, h, w = p["out"], 1, 1
    return c, h, w


def work(case):
    size, n = (2 if case["dtype"] == "bf16" else 4), case["batch"]
    if case["path"] in ("net", "module"):
        layers, shape = _structure(case)
        tot = {"flops": 0.0, "weights": 0}
        c, h, w = _walk(layers, shape, tot)
        out = n * c * h * w * (4 if layers[-1][0] == "softmax" else size)
        return {"bytes": size * (n * shape[0] * shape[1] * shape[2] + tot["weights"]) + out, "flops": n * tot["flops"]}
    if case["path"] == "conv":
        p, q = _conv_out(case)
        weights = case["k"] * case["c"] * case["r"] ** 2
        return {"bytes": size * (n * case["c"] * case["h"] * case["w"] + weights + n * case["k"] * p * q), "flops": 2.0 * n * p * q * weights}
    # fit: forward and parameter gradient; input and target in, filters in and out, gradients out
    pixels, weights = n * (case["h"] // 2) * (case["w"] // 2), case["k"] * case["c"] * 9
    return {"bytes": 4 * (n * case["c"] * case["h"] * case["w"] + pixels * case["k"] + 3 * weights), "flops": 2 * 2.0 * pixels * weights}


def tolerance(case):
    if case["path"] == "fit":
        # 32-bit sums; a pre-activation within rounding of zero may land on the other side of the ReLU, which moves the
        # gradient of its filter by one pixel's share
        return {"rel": 1e-4, "max": 1e-2}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    if case.get("net") == "googlenet":
        # about 25 roundings to bf16 on the deepest path move a logit by 0.3 % of the logits' rms; the softmax turns an
        # absolute difference of two logits into a relative one of two probabilities (1.2 to 1.7 % against fp64)
        return {"rel": 2.5e-2, "max": 0.3}
    if case.get("net") == "resnet_conv2_x":
        # up to 21 roundings: the worst of 1e8 outputs is 4 % off
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 1e-2, "max": 5e-2}
