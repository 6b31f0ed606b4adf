"""The work a user of this framework has it do, as cases that can be timed and compared.

Four kinds, all through the public entry points of `paper_1811_01532_amd`:

* ``step``    -- one replica's whole training step (`StepPlan.run`): forward, loss, backward, SGD.  What the framework
                 is for; run at per-GPU minibatches from a few images (a global minibatch divided over many GPUs) to 256.
* ``forward`` -- the forward pass alone, layer by layer, with trained weights in hand: evaluation and serving.
* ``conv``    -- one convolution block (convolution, ReLU, optionally a max-pool) forward and backward through the
                 per-operation calls: what a table of per-layer times is made of, and how a network that the step plan
                 does not know is built.
* ``fc``      -- one fully-connected layer forward and backward, also as the slice of it that one GPU of a
                 model-parallel head holds (out_features / d, rarely a round number).
"""
import math

import torch

import paper_1811_01532_amd as wap

IMAGE, CLASSES = 224, 1000

# name, input channels, output channels, filter side, stride, pad, (window, stride) of the max-pool behind it
ALEXNET_CONVS = [
    ("conv1", 3, 64, 11, 4, 2, (3, 2)), ("conv2", 64, 192, 5, 1, 2, (3, 2)), ("conv3", 192, 384, 3, 1, 1, None),
    ("conv4", 384, 256, 3, 1, 1, None), ("conv5", 256, 256, 3, 1, 1, (3, 2)),
]
VGG16_CONVS = [
    ("conv%d_%d" % (b + 1, j + 1), (3 if b == 0 else (64, 128, 256, 512, 512)[b - 1]) if j == 0 else k, k, 3, 1, 1,
     (2, 2) if j == n - 1 else None)
    for b, (k, n) in enumerate([(64, 2), (128, 2), (256, 3), (512, 3), (512, 3)]) for j in range(n)
]
NETS = {"alexnet": ALEXNET_CONVS, "vgg16": VGG16_CONVS}
FC_WIDTHS = [("fc6", 4096), ("fc7", 4096), ("fc8", CLASSES)]
# Late in a schedule: the thousands of passes that a measurement makes on one state are then all ordinary training
# steps (at the benchmark's 0.001 a fixed batch is learned by heart within some dozens and the gradients die out).
LEARNING_RATE = 0.00001


def listed():
    return [
        # a global minibatch divided over many GPUs: few images each, bound by launches and by the weights' traffic
        {"name": "alexnet_step_8", "kind": "step", "net": "alexnet", "minibatch": 8, "bias": False, "store_grads": False},
        # the AlexNet-style network at the minibatch of its committed profile
        {"name": "alexnet_step_32", "kind": "step", "net": "alexnet", "minibatch": 32, "bias": False, "store_grads": False},
        # a data-parallel replica whose share is not a power of two: gradients stored for the exchange, biases trained
        {"name": "alexnet_step_100_replica", "kind": "step", "net": "alexnet", "minibatch": 100, "bias": True, "store_grads": True},
        # VGG-16's global minibatch of 64 over eight GPUs
        {"name": "vgg16_step_8", "kind": "step", "net": "vgg16", "minibatch": 8, "bias": False, "store_grads": False},
        # the benchmark's headline step
        {"name": "vgg16_step_64", "kind": "step", "net": "vgg16", "minibatch": 64, "bias": False, "store_grads": False},
        # the third part of 64 images, rounded up, as a data-parallel replica with biases
        {"name": "vgg16_step_22_replica", "kind": "step", "net": "vgg16", "minibatch": 22, "bias": True, "store_grads": True},
        # the largest per-GPU minibatch of the benchmark's sweep
        {"name": "vgg16_step_256", "kind": "step", "net": "vgg16", "minibatch": 256, "bias": False, "store_grads": False},
        # serving one image: latency, every launch counts
        {"name": "alexnet_forward_1", "kind": "forward", "net": "alexnet", "minibatch": 1, "bias": True},
        # the small single-layer configuration (32 x 32 images, 3 to 16 channels): the smallest calls there are
        {"name": "conv_small_c3", "kind": "conv", "N": 4, "H": 32, "W": 32, "C": 3, "K": 16, "R": 3, "stride": 1, "pad": 1,
         "pool": 0, "bias": True, "x_relu": False},
        # a first layer in the per-layer table: all three passes, the gradient with respect to the image among them
        {"name": "conv_first_image_grad", "kind": "conv", "N": 24, "H": 224, "W": 224, "C": 3, "K": 64, "R": 3, "stride": 1,
         "pad": 1, "pool": 0, "bias": False, "x_relu": False},
        # a strided block of another network: odd map, channel counts that no tile divides, overlapping pool
        {"name": "conv_stride2_odd", "kind": "conv", "N": 12, "H": 57, "W": 57, "C": 72, "K": 200, "R": 3, "stride": 2,
         "pad": 1, "pool": 3, "bias": True, "x_relu": True},
        # half of the 1000-way classifier on each of two GPUs, at a minibatch that fills no tile
        {"name": "fc8_half_96", "kind": "fc", "B": 96, "n_in": 4096, "n_out": 500, "relu": False, "bias": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: mostly a multiple of 64 or 32, as networks have them, else of 8, now and then any number."""
    c = _log_int(rng, lo, hi)
    unit = rng.choice([64, 64, 64, 32, 32, 8, 8, 1])
    return max(lo, min(hi, max(1, round(c / unit)) * unit))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "forward", "conv", "conv", "conv", "conv", "fc", "fc"])
    if kind == "step":
        net = rng.choice(["alexnet", "vgg16"])
        replica = rng.random() < 0.4
        return {"kind": kind, "net": net, "minibatch": _log_int(rng, 3, 300 if net == "alexnet" else 200),
                "bias": replica and rng.random() < 0.7, "store_grads": replica}
    if kind == "forward":
        return {"kind": kind, "net": rng.choice(["alexnet", "vgg16"]), "minibatch": _log_int(rng, 1, 64), "bias": rng.random() < 0.7}
    if kind == "fc":
        out = rng.choice([_log_int(rng, 100, 4096), rng.choice([4096, 1000, 512]) // rng.choice([1, 2, 4, 8])])
        return {"kind": kind, "B": _log_int(rng, 4, 320), "n_in": rng.choice([25088, 9216, 4096, 4096, 64 * rng.randint(8, 200), rng.randint(500, 5000)]),
                "n_out": out, "relu": rng.random() < 0.5, "bias": rng.random() < 0.7}
    if rng.random() < 0.3:  # a first layer
        R = rng.choice([3, 3, 5, 7, 11])
        c = {"H": rng.choice([32, 96, 160, 192, 224, rng.randint(30, 230)]), "C": 3, "K": rng.choice([16, 32, 64, 64, 96]), "R": R,
             "stride": {3: 1, 5: 2, 7: 2, 11: 4}[R], "pad": {3: 1, 5: 2, 7: 3, 11: 2}[R], "x_relu": False}
        c["W"] = c["H"]
    else:
        R = rng.choice([1, 3, 3, 3, 3, 5])
        c = {"H": _log_int(rng, 7, 112), "C": _channels(rng, 16, 512), "K": _channels(rng, 16, 512), "R": R,
             "stride": rng.choice([1, 1, 1, 2]), "pad": R // 2, "x_relu": rng.random() < 0.7}
        c["W"] = c["H"] if rng.random() < 0.7 else _log_int(rng, 7, 112)
    c["pool"] = rng.choice([0, 0, 2, 3])
    c["bias"] = rng.random() < 0.5
    P, Q = _conv_out(c["H"], c), _conv_out(c["W"], c)
    if min(P, Q) < 4:
        c["pool"] = 0
    most = min(64, int(4e11 / (2.0 * P * Q * c["K"] * c["C"] * R * R)), int(1.5e8 / (P * Q * c["K"])), int(1.5e8 / (c["H"] * c["W"] * c["C"])))
    return {"kind": kind, "N": _log_int(rng, 1, max(1, most)), **c}


def _conv_out(n, c):
    return (n + 2 * c["pad"] - c["R"]) // c["stride"] + 1


# ---- inputs --------------------------------------------------------------------------------------------------------
class _Random:
    """Tensors on the GPU from one seed: images and gradients ~ N(0, 1), weights ~ N(0, 2 / fan_in)."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1000003 * int(seed) + 181101532)

    def f32(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32).mul_(std)

    def bf16(self, *shape, std=1.0):
        return self.f32(*shape, std=std).to(torch.bfloat16)

    def labels(self, n):
        return torch.randint(0, CLASSES, (n,), generator=self.g, device="cuda", dtype=torch.int32)


def _empty(shape, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def _layers(net, image=IMAGE):
    """(name, C, K, R, stride, pad, pool, input side, output side) of every convolution, and the first FC layer's inputs."""
    out, h = [], image
    for name, C, K, R, st, pad, pool in NETS[net]:
        p = (h + 2 * pad - R) // st + 1
        out.append((name, C, K, R, st, pad, pool, h, p))
        h = (p - pool[0]) // pool[1] + 1 if pool else p
    return out, h * h * NETS[net][-1][2]


def _prepare_step(case, rnd):
    flags = (wap.WAP_STEP_BIAS if case["bias"] else 0) | (wap.WAP_STEP_STORE_GRADS if case["store_grads"] else 0)
    plan = wap.StepPlan(case["net"], case["minibatch"], lr=LEARNING_RATE, image=IMAGE, flags=flags)
    arena = torch.empty(plan.arena_bytes(), dtype=torch.uint8, device="cuda")
    where = plan.tensors()

    def view(name, dtype):
        off, nb = where[name]
        return arena[off:off + nb].view(dtype)

    w32, w = view("params.w32", torch.float32), view("params.w", torch.bfloat16)
    w32.zero_()
    view("params.dw", torch.float32).zero_()
    layers, n_in = _layers(case["net"])
    fan_in = {name: C * R * R for name, C, K, R, *_ in layers}
    for name, width in FC_WIDTHS:
        fan_in[name] = n_in
        n_in = width
    for name, n in fan_in.items():
        t = view(name + ".w32", torch.float32)
        t.normal_(generator=rnd.g).mul_(math.sqrt(2.0 / n))
        if case["bias"]:
            view(name + ".b32", torch.float32).normal_(generator=rnd.g).mul_(0.01)
    wap.wap_cast_f32_bf16(w32.numel(), w32, w)
    view("input", torch.bfloat16).copy_(rnd.bf16(case["minibatch"] * IMAGE * IMAGE * 3))
    view("labels", torch.int32).copy_(rnd.labels(case["minibatch"]))
    out = {"loss": view("loss", torch.float32)[:1], "row_loss": view("row_loss", torch.float32),
           "logits": view("fc8.y", torch.bfloat16), "w32": w32, "w": w}
    if case["store_grads"]:
        # of the stored gradients, the classifier's: in the layers below, two correct implementations differ by 5 to 30 %
        # (bf16 roundings flip ReLU masks and pool maxima of the untrained network), which says nothing about either
        out["fc8_dw"] = view("fc8.dw", torch.float32)
        if case["bias"]:
            out["fc8_db"] = view("fc8.db", torch.float32)
    return {"plan": plan, "arena": arena, "out": out}


def _run_step(s):
    s["plan"].run(s["arena"])
    return s["out"]


def _prepare_forward(case, rnd):
    B = case["minibatch"]
    layers, n_in = _layers(case["net"])
    ops, need = [], 0
    for name, C, K, R, st, pad, pool, h, p in layers:
        d = wap.conv_desc(B, h, h, C, K, R, R, st, pad, relu=True)
        op = {"kind": "conv", "desc": d, "w": rnd.bf16(K, R, R, C, std=math.sqrt(2.0 / (C * R * R))),
              "b": rnd.f32(K, std=0.01) if case["bias"] else None, "y": _empty((B, p, p, K)), "pool": 0}
        if pool:
            q = (p - pool[0]) // pool[1] + 1
            op.update(pool=pool[0], dims=(B, p, p, K) + pool, yp=_empty((B, q, q, K)), am=_empty((B, q, q, K), torch.uint8))
            if pool == (2, 2):
                if wap.wap_conv2d_fwd_pool2x2_fused(d):
                    op["y"] = None
                need = max(need, wap.wap_conv2d_workspace_bytes(d, wap.WAP_PASS_FWD))
        ops.append(op)
    for name, width in FC_WIDTHS:
        d = wap.fc_desc(B, n_in, width, relu=name != "fc8")
        ops.append({"kind": "fc", "desc": d, "w": rnd.bf16(width, n_in, std=math.sqrt(2.0 / n_in)),
                    "b": rnd.f32(width, std=0.01) if case["bias"] else None, "y": _empty((B, width))})
        need = max(need, wap.wap_fc_workspace_bytes(d, wap.WAP_PASS_FWD))
        n_in = width
    return {"ops": ops, "ws": _workspace(need), "x": rnd.bf16(B, IMAGE, IMAGE, 3)}


def _run_forward(s):
    x, ws, features = s["x"], s["ws"], None
    for op in s["ops"]:
        if op["kind"] == "fc":
            if features is None:
                features = x
            wap.wap_fc_fwd(op["desc"], x, op["w"], op["b"], op["y"], ws)
            x = op["y"]
        elif op["pool"] == 2:
            wap.wap_conv2d_fwd_pool2x2(op["desc"], x, op["w"], op["b"], op["y"], op["yp"], op["am"], ws)
            x = op["yp"]
        else:
            wap.wap_conv2d_fwd_static_ws(op["desc"], x, op["w"], op["b"], op["y"])
            x = op["y"]
            if op["pool"]:
                wap.wap_maxpool_fwd(*op["dims"], x, op["yp"], op["am"])
                x = op["yp"]
    return {"features": features, "logits": x}


def _prepare_conv(c, rnd):
    N, H, W, C, K, R = (c[k] for k in ("N", "H", "W", "C", "K", "R"))
    P, Q = _conv_out(H, c), _conv_out(W, c)
    d = wap.conv_desc(N, H, W, C, K, R, R, c["stride"], c["pad"], relu=True)
    s = {"d": d, "w": rnd.bf16(K, R, R, C, std=math.sqrt(2.0 / (C * R * R))), "x": rnd.bf16(N, H, W, C), "x_relu": c["x_relu"],
         "b": rnd.f32(K, std=0.01) if c["bias"] else None, "y": _empty((N, P, Q, K)), "dx": _empty((N, H, W, C)),
         "dw": _empty((K, R, R, C), torch.float32), "pool": c["pool"], "fused_pool": False}
    if c["x_relu"]:
        s["x"].clamp_(min=0)
    need = max(wap.wap_conv2d_workspace_bytes(d, p) for p in (wap.WAP_PASS_FWD, wap.WAP_PASS_BWD_DATA, wap.WAP_PASS_BWD_WEIGHT))
    rows, out = N * P * Q, (N, P, Q, K)
    if c["pool"]:
        out = (N, (P - c["pool"]) // 2 + 1, (Q - c["pool"]) // 2 + 1, K)
        s.update(yp=_empty(out), am=_empty(out, torch.uint8))
        s["fused_pool"] = c["pool"] == 2 and P % 2 == 0 and Q % 2 == 0
    if s["fused_pool"]:
        rows = N * (P // 2) * (Q // 2)
        routed = all(wap.wap_conv2d_bwd_pool2x2_fused(d, p) for p in (wap.WAP_PASS_BWD_DATA, wap.WAP_PASS_BWD_WEIGHT))
        if wap.wap_conv2d_fwd_pool2x2_fused(d):
            s["y"] = None
        s["dy"] = None if routed else _empty((N, P, Q, K))
    else:
        s["dy"] = _empty((N, P, Q, K))
    s["g"], s["gm"], s["rows"] = rnd.bf16(*out), _empty(out), rows
    if c["bias"]:
        s["db"] = _empty((K,), torch.float32)
        need = max(need, wap.wap_bias_grad_workspace_bytes(rows, K))
    s["ws"] = _workspace(need)
    return s


def _run_conv(s):
    d, ws = s["d"], s["ws"]
    if s["fused_pool"]:  # the pooled gradient carries the ReLU derivative, the backward calls route it to the maxima
        wap.wap_conv2d_fwd_pool2x2(d, s["x"], s["w"], s["b"], s["y"], s["yp"], s["am"], ws)
        wap.wap_relu_bwd(s["g"], s["yp"], s["gm"], s["g"].numel())
        wap.wap_conv2d_bwd_data_pool2x2(d, s["gm"], s["am"], s["w"], s["x"] if s["x_relu"] else None, s["dx"], s["dy"], ws)
        wap.wap_conv2d_bwd_weight_pool2x2(d, s["x"], s["gm"], s["am"], s["dw"], s["dy"], ws)
        grad = s["gm"]
    else:
        wap.wap_conv2d_fwd(d, s["x"], s["w"], s["b"], s["y"], ws)
        if s["pool"]:
            wap.wap_maxpool_fwd(d.N, d.P, d.Q, d.K, s["pool"], 2, s["y"], s["yp"], s["am"])
            wap.wap_maxpool_bwd(d.N, d.P, d.Q, d.K, s["pool"], 2, s["g"], s["am"], s["yp"], s["dy"])
        else:
            wap.wap_relu_bwd(s["g"], s["y"], s["dy"], s["dy"].numel())
        if s["x_relu"]:
            wap.wap_conv2d_bwd_data_relu(d, s["dy"], s["w"], s["x"], s["dx"], ws)
        else:
            wap.wap_conv2d_bwd_data(d, s["dy"], s["w"], s["dx"], ws)
        wap.wap_conv2d_bwd_weight(d, s["x"], s["dy"], s["dw"], ws)
        grad = s["dy"]
    out = {"y": s["yp"] if s["pool"] else s["y"], "dx": s["dx"], "dw": s["dw"]}
    if s["pool"]:
        out["argmax"] = s["am"]
    if s["b"] is not None:
        wap.wap_bias_grad(s["rows"], d.K, grad, s["db"], ws)
        out["db"] = s["db"]
    return out


def _prepare_fc(c, rnd):
    B, n_in, n_out = c["B"], c["n_in"], c["n_out"]
    d = wap.fc_desc(B, n_in, n_out, relu=c["relu"])
    s = {"d": d, "w": rnd.bf16(n_out, n_in, std=math.sqrt(2.0 / n_in)), "x": rnd.bf16(B, n_in).clamp_(min=0), "g": rnd.bf16(B, n_out),
         "b": rnd.f32(n_out, std=0.01) if c["bias"] else None, "y": _empty((B, n_out)), "gm": _empty((B, n_out)),
         "dx": _empty((B, n_in)), "dw": _empty((n_out, n_in), torch.float32)}
    need = max(wap.wap_fc_workspace_bytes(d, p) for p in (wap.WAP_PASS_FWD, wap.WAP_PASS_BWD_DATA, wap.WAP_PASS_BWD_WEIGHT))
    if c["bias"]:
        s["db"] = _empty((n_out,), torch.float32)
        need = max(need, wap.wap_bias_grad_workspace_bytes(B, n_out))
    s["ws"] = _workspace(need)
    return s


def _run_fc(s):
    d, g = s["d"], s["g"]
    wap.wap_fc_fwd(d, s["x"], s["w"], s["b"], s["y"], s["ws"])
    if d.flags & wap.WAP_RELU:
        wap.wap_relu_bwd(g, s["y"], s["gm"], g.numel())
        g = s["gm"]
    wap.wap_fc_bwd(d, s["x"], s["w"], g, s["dx"], s["dw"], s["ws"])
    out = {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    if s["b"] is not None:
        wap.wap_bias_grad(d.B, d.out_features, g, s["db"], s["ws"])
        out["db"] = s["db"]
    return out


def prepare(case, seed):
    """The inputs, weights, plan and buffers a user's program holds before the call."""
    make = {"step": _prepare_step, "forward": _prepare_forward, "conv": _prepare_conv, "fc": _prepare_fc}[case["kind"]]
    return {"run": {"step": _run_step, "forward": _run_forward, "conv": _run_conv, "fc": _run_fc}[case["kind"]],
            **make(case, _Random(seed))}


def run(state):
    return state["run"](state)


def work(case):
    """Operations: two per multiply-add of every product (forward, data gradient, weight gradient; no image gradient in a
    step).  Bytes: operands and results once; in a step every weight is read and written as fp32 and as bf16 and every
    activation that the backward pass needs is written and read."""
    if case["kind"] in ("step", "forward"):
        B, train = case["minibatch"], case["kind"] == "step"
        layers, n_in = _layers(case["net"])
        flops, params, acts = 0.0, 0, B * IMAGE * IMAGE * 3
        for i, (name, C, K, R, st, pad, pool, h, p) in enumerate(layers):
            f = 2.0 * B * p * p * K * C * R * R
            flops += (f if not train else 2.0 * f if i == 0 else 3.0 * f)
            params += K * C * R * R
            q = (p - pool[0]) // pool[1] + 1 if pool else p
            acts += B * q * q * K
        for name, width in FC_WIDTHS:
            flops += (3.0 if train else 1.0) * 2.0 * B * n_in * width
            params += n_in * width
            acts += B * width
            n_in = width
        if not train:
            return {"bytes": 2.0 * params + 2.0 * B * (IMAGE * IMAGE * 3 + CLASSES), "flops": flops}
        return {"bytes": (16.0 if case["store_grads"] else 12.0) * params + 4.0 * acts, "flops": flops}
    if case["kind"] == "fc":
        x, w, y = case["B"] * case["n_in"], case["n_in"] * case["n_out"], case["B"] * case["n_out"]
        return {"bytes": 2.0 * (2 * x + w + 2 * y) + 4.0 * w, "flops": 6.0 * case["B"] * w}
    P, Q = _conv_out(case["H"], case), _conv_out(case["W"], case)
    x, y = case["N"] * case["H"] * case["W"] * case["C"], case["N"] * P * Q * case["K"]
    w = case["K"] * case["C"] * case["R"] ** 2
    g = y
    if case["pool"]:
        g = case["N"] * ((P - case["pool"]) // 2 + 1) * ((Q - case["pool"]) // 2 + 1) * case["K"]
    return {"bytes": 2.0 * (2 * x + w + 2 * g) + 4.0 * w + (g if case["pool"] else 0), "flops": 6.0 * case["N"] * P * Q * w}


def tolerance(case):
    """About four times what the same code shows with its sums in another order (other tile kernels, other reduction
    splits).  A deep ReLU network in bf16 amplifies a changed rounding: logits differ by up to 0.9 % after two steps, the
    classifier's gradient by 0.7 % (a few elements by a quarter of its RMS).  One layer: a rounding of a bf16 result in
    some thousands changes (2.5e-5), fp32 gradients differ by 1e-6, and where a changed rounding flips a ReLU mask, its
    backward results by 3e-4 (single elements by 9 % of the RMS)."""
    if case["kind"] == "step":
        return {"rel": 0.03, "max": 0.99 if case["store_grads"] else 0.15}
    if case["kind"] == "forward":
        return {"rel": 0.03, "max": 0.12}
    return {"rel": 0.0012, "max": 0.35, "differ": 0.001}
