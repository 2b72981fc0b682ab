"""The work a user of this library has it do, as timed cases.

A case is one pass through a public entry point: a whole protected network
(``CtcNet.forward``) or one protected convolution
(``ctc_conv2d_forward``).  Sizes are those of the repository's workloads
(32x32 and 224x224 networks, their layers, the widths append mode gives
them) and of the batches and image sizes around them.

Inputs are drawn on the GPU from the seed.  Convolution inputs look like the
activations the path sees: rectified values, the incoming checksum in the
last channel, filters that ignore it and a last filter that carries it on.
"""

import math

import torch
import torch.nn.functional as F

import paper_2609_16742_amd as P
from paper_2609_16742_amd import ctc
from workloads import nets

BN_EPS = 1e-5
NET_DTYPES = {"tiny": ("f32",), "resnet20": ("f32",),
              "resnet18": ("f16", "f32"), "vgg16": ("f16",),
              "mobilenetv2": ("f16",)}
# Largest batch a workload runs, and the smallest image a network takes.
NET_BATCH = {"tiny": 64, "resnet20": 128, "resnet18": 64, "vgg16": 32,
             "mobilenetv2": 128}
NET_MIN_HW = {"resnet18": 64, "vgg16": 64, "mobilenetv2": 64}


# ------------------------------------------------------------------- cases

def _net(name, net, dtype, batch, hw, protect="replace"):
    return dict(name=name, kind="net", net=net, dtype=dtype, batch=batch,
                hw=hw, protect=protect)


def _conv(name, dtype, batch, h, w, c_in, c_out, k, stride=1, depthwise=False,
          residual=False, relu=True, pool=0):
    return dict(name=name, kind="conv", dtype=dtype, batch=batch, h=h, w=w,
                c_in=c_in, c_out=c_out, k=k, stride=stride,
                depthwise=depthwise, residual=residual, relu=relu, pool=pool)


def listed():
    return [
        # The smallest call: one 32x32 image, a handful of dependent kernels.
        _net("tiny_f32_b1", "tiny", "f32", 1, 32),
        # One image at a time through a 21-layer network: a serving call,
        # where every layer has too little work for the chip.
        _net("resnet18_f16_b1", "resnet18", "f16", 1, 224),
        # CIFAR-sized network at its evaluation batch, fp32.
        _net("resnet20_f32_b128", "resnet20", "f32", 128, 32),
        # Depthwise / pointwise network at its evaluation batch.
        _net("mobilenetv2_f16_b128", "mobilenetv2", "f16", 128, 224),
        # The largest network, the benchmark's default.
        _net("vgg16_f16_b32", "vgg16", "f16", 32, 224),
        # VGG-16's third stage: most of that network's work.
        _conv("conv3x3_f16_256_56x56_b32", "f16", 32, 56, 56, 256, 256, 3),
        # The convs that close a residual block in ResNet-18's second and
        # third stages.
        _conv("conv3x3_f16_128_28x28_b64", "f16", 64, 28, 28, 128, 128, 3,
              residual=True),
        _conv("conv3x3_f16_256_14x14_b64", "f16", 64, 14, 14, 256, 256, 3,
              residual=True),
        # The same layer of the fp32 network.
        _conv("conv3x3_f32_128_28x28_b64", "f32", 64, 28, 28, 128, 128, 3,
              residual=True),
        # MobileNetV2's last conv, and the depthwise conv of its second
        # stage (as an op of its own: the networks fuse it).
        _conv("conv1x1_f16_320_1280_7x7_b128", "f16", 128, 7, 7, 320, 1280,
              1),
        _conv("dw3x3_f16_144_56x56_b128", "f16", 128, 56, 56, 144, 144, 3,
              depthwise=True),
        # Widths of append mode (one more channel, rounded up to a vector)
        # on a map that no tile divides.
        _conv("conv3x3_f16_72_136_57x53_b24", "f16", 24, 57, 53, 72, 136, 3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        case = _draw_net(rng) if rng.random() < 0.4 else _draw_conv(rng)
        w = work(case)
        # no dearer than the largest listed case: fp32 matrix work runs at
        # a sixteenth of the fp16 rate
        if (w["flops"] * (8 if case["dtype"] == "f32" else 1) < 9e11
                and w["bytes"] < 1e9):
            del case["name"]
            return case


def _draw_net(rng):
    net = rng.choice(["tiny", "resnet20", "resnet18", "resnet18", "vgg16",
                      "mobilenetv2", "mobilenetv2"])
    hw = 32
    if net in NET_MIN_HW:
        hw = rng.choice([224, rng.randint(NET_MIN_HW[net], 224)])
        if net == "vgg16":
            hw -= hw % 32                 # five pools, then a flatten
    return _net("", net, rng.choice(NET_DTYPES[net]),
                _log(rng, 1, NET_BATCH[net]), hw,
                rng.choice(["replace", "replace", "replace", "append"]))


def _draw_conv(rng):
    dtype = rng.choice(["f16", "f16", "f32"])
    vec = 8 if dtype == "f16" else 4
    k = rng.choice([1, 3, 3])
    stride = rng.choice([1, 1, 1, 2])
    h = _log(rng, 7, 112)
    w = rng.choice([h, h, max(7, h + rng.randint(-5, 5))])
    c_in = max(vec, _log(rng, 16, 1024) // vec * vec)
    batch = _log(rng, 1, 128)
    if rng.random() < 0.25:
        return _conv("", dtype, batch, h, w, c_in, c_in, 3, stride,
                     depthwise=True)
    c_out = max(vec, _log(rng, 16, 1024) // vec * vec)
    return _conv("", dtype, batch, h, w, c_in, c_out, k, stride,
                 residual=rng.random() < 0.4, relu=rng.random() < 0.8)


def _out_hw(case):
    pad = case["k"] // 2
    p = (case["h"] + 2 * pad - case["k"]) // case["stride"] + 1
    q = (case["w"] + 2 * pad - case["k"]) // case["stride"] + 1
    return p, q


def _elem(case):
    return 2 if case["dtype"] == "f16" else 4


def work(case):
    n, e = case["batch"], _elem(case)
    if case["kind"] == "conv":
        p, q = _out_hw(case)
        cg = 1 if case["depthwise"] else case["c_in"]
        wts = case["c_out"] * cg * case["k"] ** 2
        outs = n * p * q * case["c_out"]
        nbytes = (n * case["h"] * case["w"] * case["c_in"] + wts
                  + outs // (4 if case["pool"] else 1)
                  + (outs if case["residual"] else 0)) * e
        return {"bytes": nbytes + 8 * case["c_out"],
                "flops": 2 * outs * cg * case["k"] ** 2}
    net = _net_desc(case)
    shp = net.shapes()
    flops = wts = 0
    for L, (c, h, w) in zip(net.layers, shp[1:]):
        if L["op"] == "conv":
            per = L["c_in"] // L["groups"] * L["k"] ** 2
            flops += 2 * n * c * h * w * per
            wts += c * per
        elif L["op"] == "fc":
            flops += 2 * n * L["in_f"] * L["out_f"]
            wts += L["in_f"] * L["out_f"]
    c, h, w = shp[0]
    return {"bytes": 4 * n * c * h * w + e * wts + 4 * n * (net.classes + 1),
            "flops": flops}


def tolerance(case):
    # about four times the distance to the 64-bit results
    if case["kind"] == "conv":
        # fp16: outputs rounded to 11 bits (2.1e-4).  fp32: sums of up to
        # some thousand products (3e-7 at 1152, growing with the length).
        if case["dtype"] == "f16":
            return {"rel": 1e-3, "max": 1e-2}
        return {"rel": 4e-6, "max": 1e-4}
    # a change of rounding in one layer travels through all that follow
    # (fp16: 1.6e-3 in MobileNetV2's logits; fp32: 1e-6 in ResNet-18's)
    if case["dtype"] == "f16":
        return {"rel": 6e-3, "max": 4e-2}
    return {"rel": 4e-6, "max": 6e-5}


# ---------------------------------------------------------------- networks

def _net_desc(case):
    kw = dict(batch=case["batch"], dtype=case["dtype"])
    if case["net"] in NET_MIN_HW:
        kw["in_hw"] = case["hw"]
    return nets.by_name(case["net"], **kw)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _params(net, g):
    """Canonical parameters as a trained network has them: He-normal
    weights, running statistics that match the activations."""
    out = []
    for L in net.layers:
        if L["op"] not in ("conv", "fc"):
            out.append(None)
            continue
        if L["op"] == "conv":
            shape = (L["c_out"], L["c_in"] // L["groups"], L["k"], L["k"])
        else:
            shape = (L["out_f"], L["in_f"])
        fan = shape[1] * (L["k"] ** 2 if L["op"] == "conv" else 1)
        gain = 1.0 if L.get("final") else 2.0

        def uni(lo, hi):
            return lo + (hi - lo) * torch.rand(shape[0], device="cuda",
                                               generator=g)
        p = {"w": torch.randn(shape, device="cuda", generator=g)
             * math.sqrt(gain / fan)}
        if L["bias"]:
            p["b"] = uni(-1.0, 1.0) / math.sqrt(fan)
        if L.get("bn"):
            p["gamma"] = uni(*((0.2, 0.5) if L["gamma_small"]
                               else (0.5, 1.5)))
            p["beta"] = uni(-0.2, 0.2)
            p["mean"] = torch.zeros(shape[0], device="cuda")
            p["var"] = torch.ones(shape[0], device="cuda")
        out.append(p)
    if any(L.get("bn") for L in net.layers):
        x = torch.randn((4,) + net.in_shape, device="cuda", generator=g)
        _forward(net, out, x, torch.float32, statistics=True)
    return out


def _conv_nhwc(x, w, k, stride, depthwise):
    """Convolution with padding k // 2 as one product per filter tap."""
    pad = k // 2
    p = (x.shape[1] + 2 * pad - k) // stride + 1
    q = (x.shape[2] + 2 * pad - k) // stride + 1
    x = F.pad(x, (0, 0, pad, pad, pad, pad))
    y = x.new_zeros((x.shape[0], p, q, w.shape[0]))
    for r in range(k):
        for s in range(k):
            t = x[:, r:r + stride * (p - 1) + 1:stride,
                  s:s + stride * (q - 1) + 1:stride]
            if depthwise:
                y += t * w[:, 0, r, s]
            else:
                y += (t.reshape(-1, t.shape[3])
                      @ w[:, :, r, s].t()).reshape(y.shape)
    return y


def _forward(net, params, x, dt, statistics=False):
    """The network in plain torch at precision dt; with `statistics`, sets
    every BN's running statistics to those of its input on the way and
    stops at the first FC."""
    acts = [x.to(dt).permute(0, 2, 3, 1)]
    for L, p in zip(net.layers, params):
        a = acts[L["inp"]]
        if L["op"] == "conv":
            y = _conv_nhwc(a, p["w"].to(dt), L["k"], L["stride"],
                           L["groups"] > 1)
            if "b" in p:
                y += p["b"].to(dt)
            if L["bn"]:
                if statistics:
                    p["mean"] = y.mean((0, 1, 2)).float()
                    p["var"] = y.var((0, 1, 2), unbiased=False).float()
                s = p["gamma"].to(dt) / torch.sqrt(p["var"].to(dt) + BN_EPS)
                y = (y - p["mean"].to(dt)) * s + p["beta"].to(dt)
            if L["residual"] >= 0:
                y = y + acts[L["residual"]]
            if L["relu"]:
                y = torch.relu(y)
        elif L["op"] == "maxpool":
            y = F.max_pool2d(a.permute(0, 3, 1, 2), L["k"], L["stride"],
                             L["pad"]).permute(0, 2, 3, 1)
        elif L["op"] == "gap":
            y = a.mean((1, 2), keepdim=True)
        else:
            if statistics:
                return None
            if a.dim() == 4:
                a = a.permute(0, 3, 1, 2).flatten(1)
            y = a @ p["w"].to(dt).t()
            if "b" in p:
                y += p["b"].to(dt)
            if L["relu"]:
                y = torch.relu(y)
        acts.append(y)
    return acts[-1]


def _protected(net, params):
    """The parameters a protected network runs with (replace mode): the last
    filter of every conv carries the checksum, the others ignore it, the
    classifier gets the neuron that sums all its inputs."""
    out = []
    for L, p in zip(net.layers, params):
        if p is None:
            out.append(None)
            continue
        p = {k: v.clone() for k, v in p.items()}
        w, fed = p["w"], L["inp"] != 0
        if L["op"] == "conv":
            c = L["k"] // 2
            if fed and L["groups"] == 1:
                w[:-1, -1] = 0
            w[-1] = 0
            if L["groups"] > 1:
                w[-1, 0, c, c] = 1
            elif L["shortcut"]:
                w[-1, -1, c, c] = 1
            elif not L["block_first"]:
                w[-1, :, c, c] = 1
            for k, v in (("b", 0), ("mean", 0), ("var", 1), ("gamma", 1),
                         ("beta", 0)):
                if k in p:
                    p[k][-1] = v
        else:
            per = 1
            if L["flatten"] is not None:
                per = L["flatten"][1] * L["flatten"][2]
            w[:, L["in_f"] - per:] = 0
            if L["final"]:
                p["w"] = torch.cat([w, torch.ones_like(w[:1])])
                p["b"] = F.pad(p["b"], (0, 1))
            else:
                w[-1] = 1
                p["b"][-1] = 0
        if net.dtype == "f16":
            p["w"] = p["w"].half()
        out.append(p)
    return out


def _images(net, n, g):
    return torch.randn((n,) + net.in_shape, device="cuda", generator=g)


def _net_inputs(case, seed):
    """(network, parameters, calibration images, images to classify); every
    eighth image is twice as bright, which the detector has to flag."""
    g, net = _gen(seed), _net_desc(case)
    params = _params(net, g)
    cal = _images(net, case["batch"], g)
    x = _images(net, case["batch"], g)
    x[7::8] *= 2
    return net, params, cal, x


def _prepare_net(case, seed):
    desc, params, cal, x = _net_inputs(case, seed)
    host = [None if p is None else {k: v.cpu().numpy() for k, v in p.items()}
            for p in params]
    net = P.CtcNet(desc.layers, desc.in_shape, desc.classes, desc.dtype, host,
                   protect=case["protect"], max_batch=case["batch"])
    samples = net.forward(cal)[:, -1].double().cpu().numpy()
    ref, tau = ctc.ctc_threshold_from_samples(samples, 0.01)
    # few samples: a threshold of twice their spread
    net.set_threshold(ref, max(2 * tau, 0.25 * abs(ref)))
    return dict(
        net=net, x=x,
        out=torch.empty((case["batch"], net.out_cols), device="cuda"),
        flags=torch.zeros(case["batch"], dtype=torch.uint8, device="cuda"))


# ------------------------------------------------------------ convolutions

def _conv_inputs(case, seed):
    g, n = _gen(seed), case["batch"]
    dt = torch.float16 if case["dtype"] == "f16" else torch.float32
    p, q = _out_hw(case)

    def acts(h, w, c):
        a = torch.randn((n, h, w, c), device="cuda", generator=g).relu_()
        a[..., -1] = a[..., :-1].sum(-1) * 0.25 + 1
        return a.to(dt)

    x = acts(case["h"], case["w"], case["c_in"])
    res = acts(p, q, case["c_out"]) if case["residual"] else None
    c, k = case["k"] // 2, case["k"]
    cg = 1 if case["depthwise"] else case["c_in"]
    w = torch.randn((case["c_out"], cg, k, k), device="cuda", generator=g)
    w *= math.sqrt(2.0 / (cg * k * k))
    if not case["depthwise"]:
        w[:, -1] = 0
    w[-1] = 0
    w[-1, :, c, c] = 1
    scale = 0.5 + torch.rand(case["c_out"], device="cuda", generator=g)
    shift = 0.1 * torch.randn(case["c_out"], device="cuda", generator=g)
    scale[-1], shift[-1] = 1.0 / math.sqrt(1.0 + BN_EPS), 0.0
    return x, w.to(dt), scale, shift, res


def _prepare_conv(case, seed):
    x, w, scale, shift, res = _conv_inputs(case, seed)
    p, q = _out_hw(case)
    groups = case["c_in"] if case["depthwise"] else 1
    desc = ctc.layer_desc(case["c_in"], case["c_out"], case["k"], case["k"],
                          case["stride"], case["k"] // 2, groups, 1,
                          ctc.CTC_ROLE_PASS if case["depthwise"]
                          else ctc.CTC_ROLE_SUM)
    dt = ctc.DTYPES[case["dtype"]]
    # [K][R][S][C]; depthwise [R][S][K]
    packed = (w[:, 0].permute(1, 2, 0) if case["depthwise"]
              else w.permute(0, 2, 3, 1)).contiguous()
    ws = ctc.ctc_conv2d_workspace_bytes(desc, dt, case["batch"], case["h"],
                                        case["w"], case["pool"])
    if case["pool"]:
        p, q = p // 2, q // 2
    return dict(
        desc=desc, dt=dt, case=case, x=x, w=packed, scale=scale, shift=shift,
        res=res, ws_bytes=ws,
        ws=torch.empty(ws, dtype=torch.uint8, device="cuda") if ws else None,
        y=torch.empty((case["batch"], p, q, case["c_out"]), dtype=x.dtype,
                      device="cuda"))


# ------------------------------------------------------- what is measured

def prepare(case, seed):
    return (_prepare_net if case["kind"] == "net" else _prepare_conv)(case,
                                                                      seed)


def run(state):
    if "net" in state:
        out, flags = state["out"], state["flags"]
        state["net"].forward(state["x"], out, flags)
        return {"logits": out[:, :-1], "checksum": out[:, -1],
                "flags": flags}
    c, y = state["case"], state["y"]
    ctc.ctc_conv2d_forward(state["desc"], state["dt"], c["batch"], c["h"],
                           c["w"], state["x"], state["w"], state["scale"],
                           state["shift"], state["res"], c["relu"], y,
                           pool=c["pool"], workspace=state["ws"],
                           ws_bytes=state["ws_bytes"])
    return {"features": y[..., :-1], "checksum": y[..., -1]}


def exact(case, seed):
    if case["kind"] == "net":
        if case["protect"] == "append":
            return None
        net, params, _, x = _net_inputs(case, seed)
        out = _forward(net, _protected(net, params), x, torch.float64)
        return {"logits": out[:, :-1], "checksum": out[:, -1], "flags": None}
    x, w, scale, shift, res = _conv_inputs(case, seed)
    y = _conv_nhwc(x.double(), w.double(), case["k"], case["stride"],
                   case["depthwise"])
    y = y * scale.double() + shift.double()
    if res is not None:
        y += res.double()
    if case["relu"]:
        y = torch.relu(y)
    if case["pool"]:
        y = F.max_pool2d(y.permute(0, 3, 1, 2), 2).permute(0, 2, 3, 1)
    return {"features": y[..., :-1], "checksum": y[..., -1]}
