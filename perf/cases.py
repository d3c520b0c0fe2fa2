"""Performance cases of the low-precision forward path: what a program built on this library has it do.

Five kinds of work, each through the public entry points of ``paper_1711_04713_amd``:

* ``stack``       ConvStack.forward: input quantize, every LPConvolution with its fused LPAct + ReLU
                  and counters, the max-pools -- one batch of images through a network.
* ``layer``       one LPConvolution on float input: lp_quantize, then lp_conv_fwd.
* ``classifier``  a chain of LPInnerProduct layers on one batch of codes: lp_fc_fwd per layer.
* ``quantize``    conversion of one float tensor: lp_range places the point, lp_quantize rounds.
* ``calibrate``   what fixing a layer's output format takes (and what stochastic rounding of
                  activations takes on every call): lp_conv_fwd to exact int64 accumulators,
                  lp_range_acc, then lp_act or lp_act_stochastic.

Everything on the path is integer arithmetic on codes, so every output is compared exactly.
"""
import math

import torch

import paper_1711_04713_amd as lp
from lp_inputs import GIGA1NET_CONV, VGG16_CONV, VGG16_FC
from paper_1711_04713_amd.stack import ConvStack

# The classifier's layer sizes as one text: K of the first layer, then every Nout.
VGG16_DIMS = "-".join(str(v) for v in [VGG16_FC[0][1]] + [n for (_, _, n, _) in VGG16_FC])

VGG16_TAIL = 4            # index of conv3_1: the 8-bit workload runs conv3_1 .. conv5_3
CALIBRATION_IMAGES = 2    # images the per-layer formats are fixed on
ROUNDINGS = {"away": lp.LP_ROUND_NEAREST_AWAY, "even": lp.LP_ROUND_NEAREST_EVEN, "stochastic": lp.LP_ROUND_STOCHASTIC}


# ------------------------------------------------------------------------------------ cases

def _stack(net, batch, size, n_act, n_w, name=None):
    return _named({"kind": "stack", "net": net, "batch": batch, "size": size, "n_act": n_act, "n_w": n_w}, name)


def _conv(kind, batch, h, w, cin, cout, k, pad, n_act, n_w, bias, rounding, name=None):
    return _named({"kind": kind, "batch": batch, "h": h, "w": w, "cin": cin, "cout": cout, "k": k, "pad": pad,
                   "n_act": n_act, "n_w": n_w, "bias": bias, "rounding": rounding}, name)


def _classifier(batch, dims, n_act, n_w, name=None):
    return _named({"kind": "classifier", "batch": batch, "dims": dims, "n_act": n_act, "n_w": n_w}, name)


def _quantize(count, n, rounding, values, name=None):
    return _named({"kind": "quantize", "count": count, "n": n, "rounding": rounding, "values": values}, name)


def _named(case, name):
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest layer anyone runs (also the smoke test's): launches and host time are all of it
        _conv("layer", 1, 16, 16, 16, 16, 3, 1, 16, 16, False, "away", "layer_16ch_batch1"),
        # a layer whose sizes divide nothing: odd image, ragged channels, a bias, a 5x5 window
        _conv("layer", 3, 75, 93, 96, 40, 5, 2, 16, 16, True, "away", "layer_ragged_5x5_bias"),
        # one image at a time: a camera feeding the network
        _stack("vgg16", 1, 224, 16, 16, "vgg16_batch1"),
        # a small odd batch: a server that takes what has arrived
        _stack("vgg16", 5, 224, 16, 16, "vgg16_batch5"),
        # throughput: the benchmark's default workload, and the largest case
        _stack("vgg16", 32, 224, 16, 16, "vgg16_batch32"),
        # the paper's 8-bit weights under 16-bit activations
        _stack("vgg16", 16, 224, 16, 8, "vgg16_w8_batch16"),
        # 8-bit weights and activations: conv3_1 .. conv5_3 with their pools
        _stack("vgg16_tail", 64, 56, 8, 8, "vgg16_tail_8bit_batch64"),
        # the paper's own network: kernel sizes 1, 3, 5, 7 and few channels
        _stack("giga1net", 32, 224, 16, 16, "giga1net_batch32"),
        # the classifier behind a full batch, and behind one image
        _classifier(256, VGG16_DIMS, 16, 16, "classifier_batch256"),
        _classifier(1, VGG16_DIMS, 16, 16, "classifier_batch1"),
        # one 8 x 224 x 224 x 64 activation tensor to codes, its format from its own range
        _quantize(8 * 224 * 224 * 64, 16, "away", "activations", "quantize_25m"),
        # conv1_2 on two images: exact accumulators, their range, stochastic rounding
        _conv("calibrate", CALIBRATION_IMAGES, 224, 224, 64, 64, 3, 1, 16, 16, False, "stochastic", "calibrate_conv1_2"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; none costs more than the largest listed one."""
    kind = rng.choice(("stack", "stack", "stack", "layer", "layer", "classifier", "classifier", "quantize", "calibrate"))
    if kind == "stack":
        net = rng.choice(("vgg16", "vgg16", "vgg16_tail", "giga1net"))
        if net == "vgg16":       # the five pools need a multiple of 32
            return _stack(net, _log_int(rng, 1, 32), 32 * rng.randint(3, 7), rng.choice((16, 16, 12)), rng.choice((16, 16, 8)))
        if net == "vgg16_tail":  # enters behind two pools, three follow
            return _stack(net, _log_int(rng, 1, 64), 8 * rng.randint(3, 7), 8, 8)
        return _stack(net, _log_int(rng, 1, 64), 224, 16, rng.choice((16, 16, 8)))
    if kind in ("layer", "calibrate"):
        top = 3e11 if kind == "layer" else 6e10   # multiplications times 2
        while True:
            k = rng.choice((1, 3, 3, 3, 5, 7))
            n_act = rng.choice((16, 16, 8))
            step = 8 if n_act > 8 else 16
            cin = step * _log_int(rng, 16 // step, 512 // step)
            case = _conv(kind, _log_int(rng, 1, 32), _log_int(rng, 8, 224), _log_int(rng, 8, 224), cin, _log_int(rng, 8, 512),
                         k, k // 2, n_act, n_act if n_act == 8 else rng.choice((16, 16, 8)), rng.random() < 0.5,
                         rng.choice(("away", "away", "stochastic")) if kind == "calibrate" else rng.choice(("away", "away", "away", "even")))
            out = case["batch"] * case["h"] * case["w"] * case["cout"]
            if 2.0 * out * cin * k * k <= top and out <= 26_000_000 and case["batch"] * case["h"] * case["w"] * cin <= 26_000_000:
                return case
    if kind == "classifier":
        n_act = rng.choice((16, 16, 8))
        dims = rng.choice((VGG16_DIMS, "%d-%d-%d" % (16 * _log_int(rng, 32, 784), _log_int(rng, 128, 4096), _log_int(rng, 10, 1000))))
        return _classifier(_log_int(rng, 1, 256), dims, n_act, n_act if n_act == 8 else rng.choice((16, 16, 8)))
    return _quantize(_log_int(rng, 1000, 8 * 224 * 224 * 64), rng.choice((16, 16, 12, 8)), rng.choice(("away", "even", "stochastic")),
                     rng.choice(("activations", "weights")))


# ----------------------------------------------------------------------------------- shapes

def _net_layers(net):
    """[(Cin, Cout, kernel size, padding, pool after)] of a network's convolution layers."""
    if net == "giga1net":
        return [(cin, cout, k, pad, pool) for (_, cin, cout, k, _, pad, pool) in GIGA1NET_CONV]
    layers = [(cin, cout, 3, 1, pool) for (_, cin, cout, _, pool) in VGG16_CONV]
    return layers[VGG16_TAIL:] if net == "vgg16_tail" else layers


def _code_bytes(n):
    return 2 if n > 8 else 1


def _ops_per_mac(n_act, n_w):
    """int8 operations an exact product takes on an 8-bit matrix unit: two per pair of 8-bit limbs."""
    return 2 * _code_bytes(n_act) * _code_bytes(n_w)


def work(case):
    """Bytes: every input (floats or codes, weights) read once, every returned tensor written once.
    flops: int8 multiplications and additions of the exact limb products."""
    kind = case["kind"]
    if kind == "quantize":
        return {"bytes": case["count"] * (4 + _code_bytes(case["n"])), "flops": 2 * case["count"]}
    xb, wb = _code_bytes(case["n_act"]), _code_bytes(case["n_w"])
    ops = _ops_per_mac(case["n_act"], case["n_w"])
    if kind == "classifier":
        dims = [int(v) for v in case["dims"].split("-")]
        weights = sum(a * b for a, b in zip(dims, dims[1:]))
        return {"bytes": weights * wb + case["batch"] * (dims[0] + dims[-1]) * xb, "flops": ops * case["batch"] * weights}
    if kind == "stack":
        h, macs, weights = case["size"], 0, 0
        layers = _net_layers(case["net"])
        for cin, cout, k, pad, pool in layers:
            h += 2 * pad - k + 1
            macs += case["batch"] * h * h * cout * cin * k * k
            weights += cout * cin * k * k
            if pool:
                h //= 2
        nbytes = case["batch"] * (case["size"] ** 2 * layers[0][0] * 4 + h * h * layers[-1][1] * xb) + weights * wb
        return {"bytes": nbytes, "flops": ops * macs}
    ho, wo = case["h"] + 2 * case["pad"] - case["k"] + 1, case["w"] + 2 * case["pad"] - case["k"] + 1
    pixels, weights = case["batch"] * ho * wo, case["cout"] * case["cin"] * case["k"] ** 2
    inputs = case["batch"] * case["h"] * case["w"] * case["cin"]
    if kind == "layer":
        nbytes = inputs * 4 + weights * wb + pixels * case["cout"] * xb
    else:
        nbytes = inputs * xb + weights * wb + pixels * case["cout"] * (8 + xb)
    return {"bytes": nbytes, "flops": ops * pixels * weights}


def tolerance(case):
    return "exact"


# -------------------------------------------------------------------------------- preparation

def _codes(x, n, rounding=lp.LP_ROUND_NEAREST_AWAY):
    """float tensor -> (codes, format), the format from the tensor's own range."""
    q, _ = lp.lp_range(x.reshape(-1), n)
    codes = torch.empty(x.shape, dtype=torch.int16 if n > 8 else torch.int8, device="cuda")
    lp.lp_quantize(x.reshape(-1), codes, q, rounding)
    return codes, q


def _bytes_buffer(size):
    return torch.empty(max(size, 16), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape, std=1.0):
        return torch.randn(shape, device="cuda", generator=gen) * std

    def activations(*shape):   # what a ReLU leaves: half of it zeros
        return normal(*shape).clamp_(min=0)

    state = {"case": case}
    return {"stack": _prepare_stack, "layer": _prepare_conv, "calibrate": _prepare_conv,
            "classifier": _prepare_classifier, "quantize": _prepare_quantize}[case["kind"]](state, case, gen, normal, activations)


def _prepare_stack(state, case, gen, normal, activations):
    layers = _net_layers(case["net"])
    weights = [normal(cout, k, k, cin, std=math.sqrt(2.0 / (cin * k * k))) for cin, cout, k, _, _ in layers]
    shape = (case["batch"], case["size"], case["size"], layers[0][0])
    # images are U(0,1); a stack that starts inside the network sees activations
    x = activations(*shape) if case["net"] == "vgg16_tail" else torch.rand(shape, device="cuda", generator=gen)
    stack = ConvStack(weights, [pool for *_, pool in layers], n_act=case["n_act"], n_w=case["n_w"],
                      pad=[pad for _, _, _, pad, _ in layers])
    stack.calibrate(x[:CALIBRATION_IMAGES])
    stack.prepare(case["batch"], case["size"], case["size"])
    state.update(x=x, stack=stack)
    return state


def _prepare_conv(state, case, gen, normal, activations):
    n, h, w, cin, cout, k, pad = (case[key] for key in ("batch", "h", "w", "cin", "cout", "k", "pad"))
    x = activations(n, h, w, cin)
    x_codes, qx = _codes(x, case["n_act"])
    w_codes, qw = _codes(normal(cout, k, k, cin, std=math.sqrt(2.0 / (cin * k * k))), case["n_w"])
    bias = qb = None
    if case["bias"]:
        bias, qb = _codes(normal(cout, std=0.1), case["n_w"])
        if qb.f > qx.f + qw.f:
            qb = lp.QFmt(qb.n, qb.n - qx.f - qw.f, qx.f + qw.f)
    d = lp.ConvDesc(n, h, w, cin, cout, k, k, 1, pad)
    packed = _bytes_buffer(lp.lp_conv_packed_bytes(d, qx, qw))
    lp.lp_conv_pack_weights(d, qx, qw, w_codes, packed)
    out = (n, h + 2 * pad - k + 1, w + 2 * pad - k + 1, cout)
    # ReLU(N(0,1)) through He-normal weights has about the input's variance: one more integer bit
    m = min(case["n_act"], qx.m + 1)
    state.update(
        d=d, x=x, x_codes=x_codes, qx=qx, qw=qw, packed=packed, bias=bias, qb=qb, qy=lp.QFmt(case["n_act"], m, case["n_act"] - m),
        y=torch.empty(out, dtype=x_codes.dtype, device="cuda"), counters=torch.zeros(2, dtype=torch.int64, device="cuda"),
        ws=_bytes_buffer(lp.lp_conv_workspace_bytes(d, qx, qw)),
        range_ws=torch.empty(lp.LP_RANGE_WORKSPACE_WORDS, dtype=torch.int64, device="cuda"), seed=1 + gen.initial_seed())
    if case["kind"] == "calibrate":
        state["acc"] = torch.empty(out, dtype=torch.int64, device="cuda")
    return state


def _prepare_classifier(state, case, gen, normal, activations):
    m = case["batch"]
    dims = [int(v) for v in case["dims"].split("-")]
    x, qx = _codes(activations(m, dims[0]), case["n_act"])
    state.update(x=x, layers=[], counters=torch.zeros(2 * (len(dims) - 1), dtype=torch.int64, device="cuda"))
    for i, (k, n) in enumerate(zip(dims, dims[1:])):
        relu = i + 2 < len(dims)
        w, qw = _codes(normal(n, k, std=0.01), case["n_w"])
        packed = _bytes_buffer(lp.lp_fc_packed_bytes(m, k, n, qx, qw))
        lp.lp_fc_pack_weights(m, k, n, qx, qw, w, packed)
        del w
        ws = _bytes_buffer(lp.lp_fc_workspace_bytes(m, k, n, qx, qw))
        # the layer's format, fixed from its accumulators on this batch
        acc = torch.empty((m, n), dtype=torch.int64, device="cuda")
        lp.lp_fc_fwd(m, k, n, x, qx, packed, qw, acc_out=acc, relu=relu, workspace=ws)
        qy, _ = lp.lp_range_acc(acc.reshape(-1), qx.f + qw.f, relu, case["n_act"])
        y = torch.empty((m, n), dtype=x.dtype, device="cuda")
        lp.lp_fc_fwd(m, k, n, x, qx, packed, qw, qy=qy, y_codes=y, relu=relu, workspace=ws)
        state["layers"].append({"k": k, "n": n, "relu": relu, "qx": qx, "qw": qw, "qy": qy, "packed": packed, "ws": ws, "y": y})
        x, qx = y, qy
    return state


def _prepare_quantize(state, case, gen, normal, activations):
    n = case["count"]
    x = activations(n) if case["values"] == "activations" else normal(n, std=0.05)
    state.update(
        x=x, codes=torch.empty(n, dtype=torch.int16 if case["n"] > 8 else torch.int8, device="cuda"),
        counters=torch.zeros(2, dtype=torch.int64, device="cuda"),
        range_ws=torch.empty(lp.LP_RANGE_WORKSPACE_WORDS, dtype=torch.int64, device="cuda"), seed=1 + gen.initial_seed())
    return state


# ------------------------------------------------------------------------------------- passes

def run(state):
    case = state["case"]
    return {"stack": _run_stack, "layer": _run_layer, "calibrate": _run_calibrate, "classifier": _run_classifier,
            "quantize": _run_quantize}[case["kind"]](state, case)


def _run_stack(state, case):
    stack = state["stack"]
    codes = stack.forward(state["x"])
    return {"codes": codes, "zero_counts": stack.zero_counts, "sat_counts": stack.sat_counts, "input_sat": stack.input_sat}


def _run_layer(state, case):
    s = state
    s["counters"].zero_()
    lp.lp_quantize(s["x"], s["x_codes"], s["qx"])
    lp.lp_conv_fwd(s["d"], s["x_codes"], s["qx"], s["packed"], s["qw"], qy=s["qy"], y_codes=s["y"], relu=True,
                   r=ROUNDINGS[case["rounding"]], bias_codes=s["bias"], qb=s["qb"], zero_count=s["counters"][0:1],
                   sat_count=s["counters"][1:2], workspace=s["ws"])
    return {"codes": s["y"], "counters": s["counters"]}


def _run_calibrate(state, case):
    s = state
    s["counters"].zero_()
    lp.lp_conv_fwd(s["d"], s["x_codes"], s["qx"], s["packed"], s["qw"], acc_out=s["acc"], bias_codes=s["bias"], qb=s["qb"],
                   workspace=s["ws"])
    f_acc = s["qx"].f + s["qw"].f
    acc = s["acc"].reshape(-1)
    qy, lost = lp.lp_range_acc(acc, f_acc, True, case["n_act"], workspace=s["range_ws"])
    if case["rounding"] == "stochastic":
        lp.lp_act_stochastic(acc, f_acc, qy, True, s["seed"], s["y"], zero_count=s["counters"][0:1], sat_count=s["counters"][1:2])
    else:
        lp.lp_act(acc, f_acc, qy, True, s["y"], ROUNDINGS[case["rounding"]], zero_count=s["counters"][0:1],
                  sat_count=s["counters"][1:2])
    return {"acc": s["acc"], "format": list(qy.astuple()), "lost": lost, "codes": s["y"], "counters": s["counters"]}


def _run_classifier(state, case):
    x, counters = state["x"], state["counters"]
    counters.zero_()
    for i, layer in enumerate(state["layers"]):
        lp.lp_fc_fwd(case["batch"], layer["k"], layer["n"], x, layer["qx"], layer["packed"], layer["qw"], qy=layer["qy"],
                     y_codes=layer["y"], relu=layer["relu"], zero_count=counters[2 * i:2 * i + 1],
                     sat_count=counters[2 * i + 1:2 * i + 2], workspace=layer["ws"])
        x = layer["y"]
    return {"codes": [layer["y"] for layer in state["layers"]], "counters": counters}


def _run_quantize(state, case):
    s = state
    s["counters"].zero_()
    q, lost = lp.lp_range(s["x"], case["n"], workspace=s["range_ws"])
    lp.lp_quantize(s["x"], s["codes"], q, ROUNDINGS[case["rounding"]], seed=s["seed"], zero_count=s["counters"][0:1],
                   sat_count=s["counters"][1:2])
    return {"format": list(q.astuple()), "lost": lost, "codes": s["codes"], "counters": s["counters"]}
