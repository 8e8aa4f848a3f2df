"""The work that users of this framework have it do, as cases that can be timed and checked.

Every case goes through the public entry points (``ops``, ``Replica``, ``SampledSoftmaxHead``) the
way a training program calls them: buffers, workspaces, variables and recorded step programs are
made once (``prepare``), and one pass (``run``) is one call or one training step on them.

Kinds of cases:

* ``step``: a whole training step of a network as a recorded program (forward, backward, SGD).
* ``block``: the same for one inception module with its input gradient.
* ``conv``: one convolution layer, forward (with bias and ReLU), backward (filter gradient, and
  input gradient with the ReLU backward and bias gradient of the layer below) or both.
* ``image``: a first layer over RGB images, forward and filter gradient.
* ``pool``: a max-pool, forward and backward (with or without the ReLU backward).
* ``fc``: a fully connected layer, forward, filter gradient and input gradient.
* ``head``: a sampled-softmax training step of a large classifier.
* ``update``: the in-place update of a network's variables.

``exact`` computes the same in float64 with plain torch, from the same bfloat16 or fp32 inputs.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_1605_08695_amd import ops
from paper_1605_08695_amd import workloads as wl
from paper_1605_08695_amd.sampled import SampledSoftmaxHead
from paper_1605_08695_amd.step import Replica

DEV = "cuda"
_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_SIZE = {"bf16": 2, "f32": 4}


# ----------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest step: one fp32 layer with its pool, batch 8 (launches and latency count)
        dict(name="step_single_f32_b8", kind="step", net="single", n=8, hw=32, cin=16, cout=32),
        # the headline step: the AlexNet-shaped convolution stack at batch 128, bf16
        dict(name="step_alexnet_b128", kind="step", net="alexnet", n=128),
        # one inception module (GoogLeNet 4c: 14 x 14 x 512, six narrow branches), batch 128
        dict(name="block_inception_14", kind="block", n=128, hw=14, cin=512, c1=128, c3r=128, c3=256, c5r=24, c5=64,
             cp=64),
        # a large 3x3 layer's forward (VGG-16 conv6: 56 x 56 x 256, batch 64)
        dict(name="conv_fwd_56x56_256", kind="conv", dirs="fwd", dtype="bf16", n=64, h=56, w=56, cin=256, cout=256,
             kh=3, kw=3, s=1, same=True, wide=0),
        # a large 3x3 layer's backward (VGG-16 conv9: 28 x 28 x 512, batch 64)
        dict(name="conv_bwd_28x28_512", kind="conv", dirs="bwd", dtype="bf16", n=64, h=28, w=28, cin=512, cout=512,
             kh=3, kw=3, s=1, same=True, wide=0),
        # a small ragged layer, both ways (Inception-v3 1x7 over 17 x 17, 160 -> 192, batch 32, into a
        # concat buffer of 768 channels)
        dict(name="conv_17x17_1x7", kind="conv", dirs="both", dtype="bf16", n=32, h=17, w=17, cin=160, cout=192,
             kh=1, kw=7, s=1, same=True, wide=768),
        # an fp32 layer, both ways (for users who train in single precision)
        dict(name="conv_f32_28x28", kind="conv", dirs="both", dtype="f32", n=16, h=28, w=28, cin=96, cout=128,
             kh=3, kw=3, s=1, same=True, wide=0),
        # a first layer over RGB images (AlexNet conv1, batch 128)
        dict(name="image_alexnet_conv1", kind="image", n=128, h=224, w=224, cout=64, k=11, s=4, pad=2),
        # a stride-1 pooling branch, forward and backward (GoogLeNet 3b, 28 x 28 x 256, batch 128)
        dict(name="pool_28x28_s1", kind="pool", dtype="bf16", n=128, h=28, w=28, c=256, k=3, s=1, pad=1, relu=False),
        # a fully connected layer (AlexNet fc6 over 6 x 6 x 256, batch 128)
        dict(name="fc6_b128", kind="fc", n=128, hw=6, cin=256, cout=4096),
        # a language-model head by sampled softmax (2560 rows of 512, 40 000 classes, 512 sampled)
        dict(name="head_sampled_40k", kind="head", n=2560, d=512, vocab=40000, m=512),
        # Adam over the variables of AlexNet with its classifier
        dict(name="update_adam_61m", kind="update", opt="adam", n=61100840),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Channel counts as networks have them: mostly multiples of 16 or 8, now and then any number."""
    c = _log(rng, lo, hi)
    u = rng.random()
    step = 1 if u < 0.08 else (8 if u < 0.4 else 16)
    return max(step, (c + step // 2) // step * step)


_KERNELS = ((1, 1), (1, 1), (3, 3), (3, 3), (3, 3), (5, 5), (1, 7), (7, 1), (1, 3), (3, 1))


def _draw_conv(rng):
    while True:
        kh, kw = rng.choice(_KERNELS)
        s = 2 if (kh, kw) == (3, 3) and rng.random() < 0.2 else 1
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        h = _log(rng, 7, 112)
        c = dict(kind="conv", dirs=rng.choice(("fwd", "bwd", "both")), dtype=dtype, n=_log(rng, 1, 128), h=h,
                 w=h if rng.random() < 0.8 else _log(rng, 7, 112), cin=_channels(rng, 16, 1280),
                 cout=_channels(rng, 16, 768), kh=kh, kw=kw, s=s, same=s == 1 or rng.random() < 0.5, wide=0)
        if rng.random() < 0.3:                 # a branch of a concat
            c["wide"] = (c["cout"] + _channels(rng, 64, 1280) + 7) // 8 * 8
        w = work(c)
        if 1e7 <= w["flops"] <= (4.5e11 if dtype == "bf16" else 5e10) and w["bytes"] <= 6e8:
            return c


def draw(rng):
    kind = rng.choice(("step", "block", "conv", "conv", "conv", "conv", "image", "pool", "pool", "fc", "head",
                       "update"))
    if kind == "step":
        if rng.random() < 0.5:
            return dict(kind="step", net="single", n=_log(rng, 1, 64), hw=_log(rng, 8, 48), cin=_channels(rng, 8, 64),
                        cout=_channels(rng, 16, 96))
        return dict(kind="step", net="alexnet", n=_log(rng, 4, 128))
    if kind == "block":
        m = rng.choice(wl.GOOGLENET_MODULES)
        cin = {"3a": 192, "3b": 256, "4a": 480, "4b": 512, "4c": 512, "4d": 512, "4e": 528, "5a": 832, "5b": 832}[m[0]]
        hw = {"3": 28, "4": 14, "5": 7}[m[0][0]]
        return dict(kind="block", n=_log(rng, 4, 128), hw=hw, cin=cin, c1=m[1], c3r=m[2], c3=m[3], c5r=m[4], c5=m[5],
                    cp=m[6])
    if kind == "conv":
        return _draw_conv(rng)
    if kind == "image":
        while True:
            k, s, pad, cout = rng.choice(((11, 4, 2, 64), (3, 1, 1, 64), (3, 2, 0, 32), (7, 2, 3, 64)))
            h = _log(rng, 64, 320)
            c = dict(kind="image", n=_log(rng, 1, 128), h=h, w=h if rng.random() < 0.7 else _log(rng, 64, 320),
                     cout=cout, k=k, s=s, pad=pad)
            if work(c)["bytes"] <= 8e8:
                return c
    if kind == "pool":
        while True:
            k, s, pad = rng.choice(((3, 1, 1), (3, 1, 1), (3, 2, 0), (2, 2, 0)))
            h = _log(rng, 7, 112)
            c = dict(kind="pool", dtype="f32" if rng.random() < 0.15 else "bf16", n=_log(rng, 1, 128), h=h,
                     w=h if rng.random() < 0.8 else _log(rng, 7, 112), c=_channels(rng, 32, 1280), k=k, s=s, pad=pad,
                     relu=s == 2 and rng.random() < 0.6)
            if 1e5 <= work(c)["bytes"] <= 6e8:
                return c
    if kind == "fc":
        hw = rng.choice((1, 1, 6, 7))
        return dict(kind="fc", n=_log(rng, 1, 256), hw=hw, cin=_channels(rng, 256, 512) if hw > 1 else
                    _channels(rng, 512, 4096), cout=rng.choice((1000, 1000, 4096, _channels(rng, 256, 4096))))
    if kind == "head":
        vocab = _log(rng, 5000, 80000)
        return dict(kind="head", n=_log(rng, 128, 4096), d=_channels(rng, 128, 1024) // 8 * 8 or 128, vocab=vocab,
                    m=_log(rng, 64, 1024))
    return dict(kind="update", opt=rng.choice(("sgd", "momentum", "adam")), n=_log(rng, 10000, 61100840))


# ----------------------------------------------------------------------------- shapes
def _conv_geom(c):
    kh, kw, s = c["kh"], c["kw"], c["s"]
    pads = wl.same_pads(c["h"], c["w"], kh, kw, s, s) if c["same"] else wl.VALID
    return pads, wl.out_len(c["h"], kh, s, pads[0], pads[1]), wl.out_len(c["w"], kw, s, pads[2], pads[3])


def _net(c):
    """The network of a step or block case.  The learning rate is small, so that the variables stay
    near their start over many steps on one batch of the surrogate loss <g, output>."""
    if c["kind"] == "step" and c["net"] == "single":
        net = wl.single_layer(batch=c["n"], hw=c["hw"], cin=c["cin"], cout=c["cout"])
    elif c["kind"] == "step":
        net = wl.alexnet(batch=c["n"])
    else:
        n, hw, cin = c["n"], c["hw"], c["cin"]
        cat = c["c1"] + c["c3"] + c["c5"] + c["cp"]
        t = {"x": (n, hw, hw, cin), "cat": (n, hw, hw, cat), "r3": (n, hw, hw, c["c3r"]), "r5": (n, hw, hw, c["c5r"]),
             "p": (n, hw, hw, cin)}
        z = (0, 0, 0, 0)
        o = [wl.Conv("b1", "x", "cat", 0, c["c1"], 1, 1, 1, 1, z),
             wl.Conv("b3r", "x", "r3", 0, c["c3r"], 1, 1, 1, 1, z),
             wl.Conv("b3", "r3", "cat", c["c1"], c["c3"], 3, 3, 1, 1, (1, 1, 1, 1)),
             wl.Conv("b5r", "x", "r5", 0, c["c5r"], 1, 1, 1, 1, z),
             wl.Conv("b5", "r5", "cat", c["c1"] + c["c3"], c["c5"], 5, 5, 1, 1, (2, 2, 2, 2)),
             wl.Pool("bp", "x", "p", 0, 3, 3, 1, 1, (1, 1, 1, 1)),
             wl.Conv("bpp", "p", "cat", c["c1"] + c["c3"] + c["c5"], c["cp"], 1, 1, 1, 1, z)]
        net = wl.Net("inception", "bf16", 0.01, True, t, o, "cat")
    return dataclasses.replace(net, lr=1e-6 if c.get("net") == "alexnet" else 1e-5)


class _Rand:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(DEV).manual_seed(int(seed))

    def normal(self, *shape, scale=1.0):
        return torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32) * scale

    def relu(self, *shape):
        return self.normal(*shape).clamp_(min=0.0)


def _net_inputs(net, seed):
    r = _Rand(seed)
    x = r.normal(*net.tensors["x"])
    if net.name == "inception":
        x.clamp_(min=0.0)                       # a module reads the ReLU outputs of the one before
    w = {c.name: r.normal(c.kh, c.kw, net.tensors[c.src][3], c.cout,
                          scale=math.sqrt(2.0 / (c.kh * c.kw * net.tensors[c.src][3]))) for c in net.convs}
    b = {c.name: r.normal(c.cout, scale=0.05) for c in net.convs}
    g = r.normal(*net.tensors[net.output], scale=1.0 / net.tensors["x"][0])
    return x, w, b, g


def _conv_inputs(c, seed):
    """x is a ReLU output, w He-normal, dy a gradient; the same values for prepare and exact."""
    r, dt = _Rand(seed), _DT[c["dtype"]]
    pads, oh, ow = _conv_geom(c)
    x = r.relu(c["n"], c["h"], c["w"], c["cin"]).to(dt)
    w = r.normal(c["kh"], c["kw"], c["cin"], c["cout"], scale=math.sqrt(2.0 / (c["kh"] * c["kw"] * c["cin"]))).to(dt)
    b = r.normal(c["cout"], scale=0.1)
    wide = c["wide"] or c["cout"]
    dy = r.normal(c["n"], oh, ow, wide).to(dt)[..., wide - c["cout"]:]
    return x, w, b, dy


def _image_inputs(c, seed):
    r = _Rand(seed)
    oh = wl.out_len(c["h"], c["k"], c["s"], c["pad"], c["pad"])
    ow = wl.out_len(c["w"], c["k"], c["s"], c["pad"], c["pad"])
    x4 = torch.zeros((c["n"], c["h"], c["w"], 4), dtype=torch.bfloat16, device=DEV)   # RGBx storage
    x4[..., :3] = r.normal(c["n"], c["h"], c["w"], 3).to(torch.bfloat16)
    w = r.normal(c["k"], c["k"], 3, c["cout"], scale=math.sqrt(2.0 / (c["k"] * c["k"] * 3))).to(torch.bfloat16)
    b = r.normal(c["cout"], scale=0.1)
    dy = r.normal(c["n"], oh, ow, c["cout"]).to(torch.bfloat16)
    return x4[..., :3], w, b, dy


def _pool_geom(c):
    return (wl.out_len(c["h"], c["k"], c["s"], c["pad"], c["pad"]),
            wl.out_len(c["w"], c["k"], c["s"], c["pad"], c["pad"]))


def _pool_inputs(c, seed):
    r, dt = _Rand(seed), _DT[c["dtype"]]
    oh, ow = _pool_geom(c)
    return r.relu(c["n"], c["h"], c["w"], c["c"]).to(dt), r.normal(c["n"], oh, ow, c["c"]).to(dt)


def _fc_inputs(c, seed):
    r, hw = _Rand(seed), c["hw"]
    x = r.relu(c["n"], hw, hw, c["cin"]).to(torch.bfloat16)
    w = r.normal(hw, hw, c["cin"], c["cout"], scale=math.sqrt(2.0 / (hw * hw * c["cin"]))).to(torch.bfloat16)
    return x, w, r.normal(c["cout"], scale=0.1), r.normal(c["n"], 1, 1, c["cout"], scale=1.0 / c["n"]).to(torch.bfloat16)


def _head_inputs(c, seed):
    rng = np.random.default_rng(seed)
    r = _Rand(seed)
    h = r.normal(c["n"], c["d"]).to(torch.bfloat16)
    W = r.normal(c["vocab"], c["d"], scale=1.0 / math.sqrt(c["d"])).cpu().numpy()
    b = r.normal(c["vocab"], scale=0.1).cpu().numpy()
    # word frequencies of a language model are Zipfian
    labels = np.minimum((np.exp(rng.random(c["n"]) * math.log(c["vocab"] + 1.0)) - 1.0).astype(np.int64),
                        c["vocab"] - 1).astype(np.int32)
    sampled, log_expected = wl.log_uniform_sample(rng, c["vocab"], c["m"])
    return h, W, b, labels, sampled, log_expected(labels), log_expected(sampled)


def _update_inputs(c, seed):
    r = _Rand(seed)
    slots = [r.normal(c["n"], scale=0.01).abs_() if i else r.normal(c["n"], scale=0.01)
             for i in range({"sgd": 0, "momentum": 1, "adam": 2}[c["opt"]])]
    return r.normal(c["n"], scale=0.02), r.normal(c["n"], scale=0.01), slots


# ----------------------------------------------------------------------------- prepare
def _workspace(nbytes):
    return torch.empty(max(16, (nbytes + 15) // 16 * 16), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    k = case["kind"]
    if k in ("step", "block"):
        net = _net(case)
        x, w, b, g = _net_inputs(net, seed)
        host = lambda t: t.cpu().numpy()                                       # noqa: E731
        rep = Replica(net, wl.Inputs(host(x), {n: host(t) for n, t in w.items()}, {n: host(t) for n, t in b.items()},
                                     host(g)), DEV)
        start = rep.snapshot()
        prog = rep.record_step()               # recording runs a step; training starts after it
        rep.restore(start)
        return dict(kind=k, rep=rep, prog=prog)
    if k == "conv":
        x, w, b, dy = _conv_inputs(case, seed)
        pads, oh, ow = _conv_geom(case)
        s = dict(kind=k, dirs=case["dirs"], x=x, w=w, b=b, dy=dy, pads=pads, s=(case["s"], case["s"]),
                 khw=(case["kh"], case["kw"]))
        need = lambda op: ops.conv2d_workspace_bytes(op, x, case["cout"], case["kh"], case["kw"],  # noqa: E731
                                                     (case["s"], case["s"]), pads)
        if case["dirs"] != "bwd":
            wide = case["wide"] or case["cout"]
            s["y"] = torch.zeros((case["n"], oh, ow, wide), dtype=x.dtype, device=DEV)[..., wide - case["cout"]:]
        if case["dirs"] != "fwd":
            s.update(dw=torch.zeros(tuple(w.shape), dtype=torch.float32, device=DEV), dpre=torch.zeros_like(x),
                     db=torch.zeros(case["cin"], dtype=torch.float32, device=DEV))
        s["ws"] = _workspace(max(need(op) for op in (0, 2, 3)))
        return s
    if k == "image":
        x, w, b, dy = _image_inputs(case, seed)
        pads = (case["pad"],) * 4
        need = max(ops.conv2d_workspace_bytes(op, x, case["cout"], case["k"], case["k"], case["s"], pads) for op in (0, 2))
        return dict(kind=k, x=x, w=w, b=b, dy=dy, s=case["s"], k=case["k"], pads=pads, ws=_workspace(need),
                    y=torch.zeros_like(dy), dw=torch.zeros(tuple(w.shape), dtype=torch.float32, device=DEV))
    if k == "pool":
        x, dy = _pool_inputs(case, seed)
        return dict(kind=k, x=x, dy=dy, k=(case["k"],) * 2, s=case["s"], pads=(case["pad"],) * 4, relu=case["relu"],
                    y=torch.zeros_like(dy), dx=torch.zeros_like(x),
                    taps=torch.zeros(tuple(dy.shape), dtype=torch.uint8, device=DEV),
                    db=torch.zeros(case["c"], dtype=torch.float32, device=DEV),
                    ws=_workspace(ops.bias_relu_bwd_workspace_bytes(x)))
    if k == "fc":
        x, w, b, dy = _fc_inputs(case, seed)
        need = max(ops.conv2d_workspace_bytes(op, x, case["cout"], case["hw"], case["hw"], 1, wl.VALID) for op in (0, 1, 2))
        return dict(kind=k, x=x, w=w, b=b, dy=dy, hw=case["hw"], ws=_workspace(need), y=torch.zeros_like(dy),
                    dw=torch.zeros(tuple(w.shape), dtype=torch.float32, device=DEV), dx=torch.zeros_like(x))
    if k == "head":
        h, W, b, labels, sampled, lq_true, lq_sampled = _head_inputs(case, seed)
        head = SampledSoftmaxHead(W, b, 0.01, DEV)
        return dict(kind=k, head=head, h=h, bt=head.prepare(labels, sampled, lq_true, lq_sampled))
    var, grad, slots = _update_inputs(case, seed)
    return dict(kind=k, opt=case["opt"], var=var, grad=grad, slots=slots, t=0,
                shadow=torch.zeros(case["n"], dtype=torch.bfloat16, device=DEV))


# ----------------------------------------------------------------------------- run
def run(state):
    k = state["kind"]
    if k in ("step", "block"):
        rep = state["rep"]
        rep.run_program(state["prog"])
        out = dict(y=rep.act[rep.net.output], W=dict(rep.W), b=dict(rep.b))
        if rep.net.input_grad:                 # a layer or block: its gradients too (see tolerance)
            out.update(dW=dict(rep.dW), db=dict(rep.db), dx=rep.grad["x"])
        return out
    if k == "conv":
        out, s = {}, state
        if s["dirs"] != "bwd":
            out["y"] = ops.conv2d_fwd_bias_relu(s["x"], s["w"], s["b"], s["s"], s["pads"], y=s["y"], ws=s["ws"])
        if s["dirs"] != "fwd":
            out["dw"] = ops.conv2d_bwd_filter(s["x"], s["dy"], s["khw"], s["s"], s["pads"], dw=s["dw"], ws=s["ws"])
            out["dpre"], out["db"] = ops.conv2d_bwd_input_relu_bwd(s["dy"], s["w"], s["x"], s["dpre"], s["s"], s["pads"],
                                                                   dbias=s["db"], ws=s["ws"])
        return out
    if k == "image":
        s = state
        y = ops.conv2d_fwd_bias_relu(s["x"], s["w"], s["b"], s["s"], s["pads"], y=s["y"], ws=s["ws"])
        dw = ops.conv2d_bwd_filter(s["x"], s["dy"], (s["k"], s["k"]), s["s"], s["pads"], dw=s["dw"], ws=s["ws"])
        return dict(y=y, dw=dw)
    if k == "pool":
        s = state
        y, taps = ops.maxpool_fwd(s["x"], s["k"], s["s"], s["pads"], y=s["y"], argmax=s["taps"], taps=True)
        if s["relu"]:
            dx, db = ops.maxpool_bwd_relu_bwd(s["dy"], taps, s["x"], s["dx"], s["k"], s["s"], s["pads"], dbias=s["db"],
                                              ws=s["ws"], py=y)
            return dict(y=y, taps=taps, dx=dx, db=db)
        return dict(y=y, taps=taps, dx=ops.maxpool_bwd(s["dy"], taps, s["dx"], s["k"], s["s"], s["pads"]))
    if k == "fc":
        s, khw = state, (state["hw"], state["hw"])
        y = ops.conv2d_fwd_bias_relu(s["x"], s["w"], s["b"], 1, wl.VALID, y=s["y"], ws=s["ws"])
        dw = ops.conv2d_bwd_filter(s["x"], s["dy"], khw, 1, wl.VALID, dw=s["dw"], ws=s["ws"])
        dx = ops.conv2d_bwd_input(s["dy"], s["w"], s["dx"], 1, wl.VALID, ws=s["ws"])
        return dict(y=y, dw=dw, dx=dx)
    if k == "head":
        loss, dh = state["head"].run(state["h"], state["bt"])
        return dict(loss=loss, dh=dh, W=state["head"].W, b=state["head"].b)
    s = state
    s["t"] += 1
    if s["opt"] == "sgd":
        ops.apply_sgd(s["var"], s["grad"], 0.01, shadow=s["shadow"])
    elif s["opt"] == "momentum":
        ops.apply_momentum(s["var"], s["slots"][0], s["grad"], 0.01, 0.9, shadow=s["shadow"])
    else:
        ops.apply_adam(s["var"], s["slots"][0], s["slots"][1], s["grad"], 1e-3, 0.9, 0.999, 1e-8, s["t"],
                       shadow=s["shadow"])
    return dict(var=s["var"], slots=s["slots"], shadow=s["shadow"])


# ----------------------------------------------------------------------------- work
def _numel(shape):
    return int(np.prod(shape))


def work(case):
    k = case["kind"]
    if k in ("step", "block"):
        net = _net(case)
        el = 4 if net.dtype == "f32" else 2
        flops = wl.conv_flops(net)
        # x and g in, the output and the input's gradient out; each tensor between is written and read
        # once in the forward pass, read again by the backward pass, and its gradient written and read
        by = _numel(net.tensors["x"]) * el * (2 + int(net.input_grad)) + 2 * _numel(net.tensors[net.output]) * el
        by += sum(5 * _numel(s) * el for t, s in net.tensors.items() if t not in ("x", net.output))
        # the filters as read by the passes, gradients written and read, variables and copies updated
        by += net.param_count() * (2 * el + 16 + (2 if el == 2 else 0))
        return dict(bytes=by, flops=flops)
    if k == "conv":
        el = _SIZE[case["dtype"]]
        pads, oh, ow = _conv_geom(case)
        nx, ny = case["n"] * case["h"] * case["w"] * case["cin"], case["n"] * oh * ow * case["cout"]
        nw = case["kh"] * case["kw"] * case["cin"] * case["cout"]
        f = 2.0 * case["n"] * oh * ow * nw
        fwd, bwd = (nx + ny + nw) * el + 4 * case["cout"], (2 * nx + ny + nw) * el + 4 * nw + 4 * case["cin"]
        d = case["dirs"]
        if d == "both":
            return dict(bytes=fwd + bwd, flops=3 * f)
        return dict(bytes=fwd if d == "fwd" else bwd, flops=f if d == "fwd" else 2 * f)
    if k == "image":
        oh = wl.out_len(case["h"], case["k"], case["s"], case["pad"], case["pad"])
        ow = wl.out_len(case["w"], case["k"], case["s"], case["pad"], case["pad"])
        nx, ny = case["n"] * case["h"] * case["w"] * 3, case["n"] * oh * ow * case["cout"]
        nw = case["k"] * case["k"] * 3 * case["cout"]
        return dict(bytes=2 * nx * 2 + 2 * ny * 2 + nw * 6, flops=4.0 * case["n"] * oh * ow * nw)
    if k == "pool":
        el = _SIZE[case["dtype"]]
        oh, ow = _pool_geom(case)
        nx, ny = case["n"] * case["h"] * case["w"] * case["c"], case["n"] * oh * ow * case["c"]
        # forward: x in, y and taps out; backward: dy and taps in (with the ReLU mask, y too), dx out
        return dict(bytes=nx * el + ny * (el + 1) + ny * (el + 1) + nx * el + (ny * el if case["relu"] else 0), flops=0)
    if k == "fc":
        kin = case["hw"] * case["hw"] * case["cin"]
        nx, ny, nw = case["n"] * kin, case["n"] * case["cout"], kin * case["cout"]
        return dict(bytes=2 * (3 * nx + 3 * ny) + nw * (2 + 4 + 2), flops=6.0 * case["n"] * nw)
    if k == "head":
        n, d, m = case["n"], case["d"], case["m"]
        # candidates: the sample and (under Zipfian labels) about half as many true classes as rows
        u = min(case["vocab"], m + n // 2)
        return dict(bytes=2 * 2 * n * d + u * d * (2 + 4 + 4 + 2) + u * 8 + 4 * n, flops=6.0 * n * d * u)
    return dict(bytes=case["n"] * {"sgd": 14, "momentum": 22, "adam": 30}[case["opt"]], flops=0)


# ----------------------------------------------------------------------------- tolerance
def tolerance(case):
    """About four times the relative error against float64 measured over listed and drawn cases
    (bf16 results 1.7e-3, fp32 sums up to 7e-7, rounded up for the longest of them; the stack's
    output 1.1e-3); in bf16 it is the rounding of results and of what the path keeps between ops."""
    k = case["kind"]
    if k == "step":
        # fp32: sums in another order.  The bf16 stack: activations that round the other way travel
        # through the layers and move the choice of a max-pool's tap or a ReLU's mask now and then; its
        # filter gradients are sums of terms of either sign (the upstream gradient is noise), where one
        # choice in a thousand shows as several per cent, so the step returns the updated variables
        # and its output, and the gradients are compared in the single layers and the block.
        return {"rel": 1e-5, "max": 1e-4} if case["net"] == "single" else {"rel": 5e-3, "max": 5e-2}
    if k == "block":
        return {"rel": 7e-3, "max": 8e-2}
    if k == "conv":
        return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 2e-2}
    if k in ("image", "fc"):
        return {"rel": 7e-3, "max": 2e-2}
    if k == "pool":
        # maxima and taps are copied; overlapping windows' gradients are summed in fp32 and rounded once
        return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 2e-2}
    if k == "head":
        return {"rel": 7e-3, "max": 0.1}       # logits and their gradient are kept in bf16
    return {"rel": 7e-3, "max": 2e-2}          # the bf16 copy; the fp32 slots move by an ulp


# ----------------------------------------------------------------------------- exact
def _rnd(t, dt):
    """Values as dt (bf16 or fp32) holds them, in float64."""
    return t.to(dt).double()


def _patches(x, kh, kw, sh, sw, pads, oh, ow, fill=0.0):
    """The (kh, kw) taps of every window of x (float64 NHWC), in scan order, as views."""
    pt, pb, pl, pr = pads
    xp = torch.nn.functional.pad(x, (0, 0, pl, pr, pt, pb), value=fill)
    for a in range(kh):
        for b in range(kw):
            yield a, b, xp[:, a:a + sh * (oh - 1) + 1:sh, b:b + sw * (ow - 1) + 1:sw, :]


def _conv64(x, w, sh, sw, pads, oh, ow):
    kh, kw, cin, cout = w.shape
    y = torch.zeros((x.shape[0] * oh * ow, cout), dtype=torch.float64, device=x.device)
    for a, b, v in _patches(x, kh, kw, sh, sw, pads, oh, ow):
        y += torch.mm(v.reshape(-1, cin), w[a, b])
    return y.view(x.shape[0], oh, ow, cout)


def _filter64(x, dy, kh, kw, sh, sw, pads):
    oh, ow, cout = dy.shape[1:]
    d = dy.reshape(-1, cout)
    dw = torch.zeros((kh, kw, x.shape[3], cout), dtype=torch.float64, device=x.device)
    for a, b, v in _patches(x, kh, kw, sh, sw, pads, oh, ow):
        dw[a, b] = torch.mm(v.reshape(-1, x.shape[3]).t().contiguous(), d)
    return dw


def _input64(dy, w, shape, sh, sw, pads):
    kh, kw, cin, cout = w.shape
    n, h, wd, _ = shape
    oh, ow = dy.shape[1:3]
    pt, pb, pl, pr = pads
    dx = torch.zeros((n, h + pt + pb, wd + pl + pr, cin), dtype=torch.float64, device=dy.device)
    d = dy.reshape(-1, cout)
    for a in range(kh):
        for b in range(kw):
            dx[:, a:a + sh * (oh - 1) + 1:sh, b:b + sw * (ow - 1) + 1:sw, :] += torch.mm(
                d, w[a, b].t().contiguous()).view(n, oh, ow, cin)
    return dx[:, pt:pt + h, pl:pl + wd, :]


def _pool64(x, k, s, pads, oh, ow):
    y = taps = None
    for a, b, v in _patches(x, k, k, s, s, pads, oh, ow, fill=-math.inf):
        if y is None:
            y, taps = v.clone(), torch.zeros(v.shape, dtype=torch.uint8, device=x.device)
            continue
        up = v > y
        y = torch.where(up, v, y)
        taps[up] = a * k + b
    return y, taps


def _unpool64(dy, taps, shape, k, s, pads):
    n, h, w, c = shape
    oh, ow = dy.shape[1:3]
    pt, pb, pl, pr = pads
    dx = torch.zeros((n, h + pt + pb, w + pl + pr, c), dtype=torch.float64, device=dy.device)
    for a in range(k):
        for b in range(k):
            dx[:, a:a + s * (oh - 1) + 1:s, b:b + s * (ow - 1) + 1:s, :] += dy * (taps == a * k + b)
    return dx[:, pt:pt + h, pl:pl + w, :]


def _net_exact(net, x, w, b, g, stored):
    """``stored``: round what the path stores between ops to the network's type.  The AlexNet stack's
    max-pools need it: unrounded, their choice of a tap differs wherever two of a window's values
    are equal in bfloat16."""
    dt = torch.float32 if net.dtype == "f32" else torch.bfloat16
    W = {n: _rnd(t, dt) for n, t in w.items()}
    B = {n: _rnd(t, dt) for n, t in b.items()}
    keep = (lambda t: _rnd(t, dt)) if stored else (lambda t: t)
    act = {t: torch.zeros(s, dtype=torch.float64, device=DEV) for t, s in net.tensors.items()}
    act["x"] = _rnd(x, dt)
    taps = {}
    for op in net.ops:
        _, oh, ow, _ = net.tensors[op.dst]
        if isinstance(op, wl.Conv):
            y = _conv64(act[op.src], W[op.name], op.sh, op.sw, op.pads, oh, ow) + B[op.name]
            act[op.dst][..., op.dst_c0:op.dst_c0 + op.cout] = keep(y.clamp_(min=0.0))
        else:
            act[op.dst], taps[op.name] = _pool64(act[op.src], op.kh, op.sh, op.pads, oh, ow)
    grad = {net.output: _rnd(g, dt)}
    dW, db = {}, {}
    for op in reversed(net.ops):
        dy = grad[op.dst]
        if isinstance(op, wl.Conv):
            sl = slice(op.dst_c0, op.dst_c0 + op.cout)
            dpre = dy[..., sl] * (act[op.dst][..., sl] > 0)
            dW[op.name] = _filter64(act[op.src], dpre, op.kh, op.kw, op.sh, op.sw, op.pads)
            db[op.name] = dpre.sum(dim=(0, 1, 2))
            if op.src == "x" and not net.input_grad:
                continue
            d = _input64(dpre, W[op.name], net.tensors[op.src], op.sh, op.sw, op.pads)
        else:
            d = _unpool64(dy, taps[op.name], net.tensors[op.src], op.kh, op.sh, op.pads)
        grad[op.src] = keep(d + grad[op.src] if op.src in grad else d)
    lr = float(np.float32(net.lr))
    out = dict(y=act[net.output], W={n: W[n] - lr * dW[n] for n in W}, b={n: B[n] - lr * db[n] for n in B})
    if net.input_grad:
        out.update(dW=dW, db=db, dx=grad["x"])
    return out


def exact(case, seed):
    k = case["kind"]
    if k in ("step", "block"):
        net = _net(case)
        return _net_exact(net, *_net_inputs(net, seed), stored=case.get("net") == "alexnet")
    if k == "conv":
        x, w, b, dy = (t.double() for t in _conv_inputs(case, seed))
        pads, oh, ow = _conv_geom(case)
        s, out = case["s"], {}
        if case["dirs"] != "bwd":
            out["y"] = (_conv64(x, w, s, s, pads, oh, ow) + b).clamp_(min=0.0)
        if case["dirs"] != "fwd":
            out["dw"] = _filter64(x, dy, case["kh"], case["kw"], s, s, pads)
            out["dpre"] = _input64(dy, w, x.shape, s, s, pads) * (x > 0)
            out["db"] = out["dpre"].sum(dim=(0, 1, 2))
        return out
    if k == "image":
        x, w, b, dy = (t.double() for t in _image_inputs(case, seed))
        pads, s = (case["pad"],) * 4, case["s"]
        return dict(y=(_conv64(x, w, s, s, pads, *dy.shape[1:3]) + b).clamp_(min=0.0),
                    dw=_filter64(x, dy, case["k"], case["k"], s, s, pads))
    if k == "pool":
        x, dy = (t.double() for t in _pool_inputs(case, seed))
        pads = (case["pad"],) * 4
        y, taps = _pool64(x, case["k"], case["s"], pads, *_pool_geom(case))
        dx = _unpool64(dy, taps, x.shape, case["k"], case["s"], pads)
        if not case["relu"]:
            return dict(y=y, taps=taps, dx=dx)
        dx = dx * (x > 0)
        return dict(y=y, taps=taps, dx=dx, db=dx.sum(dim=(0, 1, 2)))
    if k == "fc":
        x, w, b, dy = (t.double() for t in _fc_inputs(case, seed))
        return dict(y=(_conv64(x, w, 1, 1, wl.VALID, 1, 1) + b).clamp_(min=0.0),
                    dw=_filter64(x, dy, case["hw"], case["hw"], 1, 1, wl.VALID),
                    dx=_input64(dy, w, x.shape, 1, 1, wl.VALID))
    if k == "head":
        h, W, b, labels, sampled, lq_true, lq_sampled = _head_inputs(case, seed)
        n, m, bf = case["n"], case["m"], torch.bfloat16
        cand, true_pos = SampledSoftmaxHead.candidates(labels, sampled)
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)       # noqa: E731
        idx, tp, rows = up(cand).long(), up(true_pos).long(), torch.arange(n, device=DEV)
        W, b, h = _rnd(up(W), bf), up(b).double(), h.double()
        z = torch.mm(h, W[idx].t().contiguous()) + b[idx]
        # the true class by its own expected count; the sampled ones by theirs, a hit left out
        zt = z[rows, tp] - up(lq_true.astype(np.float32)).double()
        z[:, :m] -= up(lq_sampled.astype(np.float32)).double()
        z[:, m:] = -math.inf
        z[rows, tp] = zt
        p = torch.softmax(z, dim=1)
        loss = torch.logsumexp(z, dim=1) - zt
        p[rows, tp] -= 1.0
        dz = p / n
        lr = float(np.float32(0.01))
        dW, db = torch.mm(dz.t().contiguous(), h), dz.sum(dim=0)
        dh = torch.mm(dz, W[idx])
        W[idx] -= lr * dW
        b[idx] -= lr * db
        return dict(loss=loss, dh=dh, W=W, b=b)
    var, grad, slots = _update_inputs(case, seed)
    var, g = var.double(), grad.double()
    f = lambda v: float(np.float32(v))                                          # noqa: E731
    s = [t.double() for t in slots]
    if case["opt"] == "sgd":
        var = var - f(0.01) * g
    elif case["opt"] == "momentum":
        s[0] = f(0.9) * s[0] + g
        var = var - f(0.01) * s[0]
    else:
        b1, b2 = f(0.9), f(0.999)
        s = [b1 * s[0] + (1 - b1) * g, b2 * s[1] + (1 - b2) * g * g]
        var = var - f(1e-3) / (1 - b1) * s[0] / (torch.sqrt(s[1] / (1 - b2)) + f(1e-8))
    return dict(var=var, slots=s, shadow=var)
