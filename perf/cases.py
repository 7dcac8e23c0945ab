"""The work a user has this library do, as cases that can be timed and compared.

Whole training runs go through ``Trainer`` (``cdp_step`` / ``cdp_drain`` / ``cdp_get_weights`` / ``cdp_get_losses``),
single layers through the kernel-level entry points (``cdp_k_gemm``, ``cdp_k_conv``, ``cdp_k_layernorm``, ``cdp_k_gelu``,
``cdp_k_attention``), each forward and backward.  ``exact`` gives the same results in 64 bits from plain torch.

A case is a dict of plain values; ``kind`` says what it is:

  train      ``steps`` steps of a model, the drain of the cyclic timeline, then the weights of all stages and the losses
  linear     a Linear layer on ``rows`` rows: forward, data gradient, weight gradient
  conv       a convolution (k = 1 on a 1 x T image: a token-wise linear map): forward, data gradient, weight gradient
  attention  the self-attention core, forward and backward
  norm_gelu  the memory-bound layers of a transformer block: LayerNorm and GELU, forward and backward
"""
import math
from collections import namedtuple

import numpy as np
import torch
import torch.nn.functional as F

from paper_2403_08837_amd import binding as cdp

Layer = namedtuple("Layer", "kind src p")
LINEAR, RELU, CONV2D, AFFINE, ADD, MAXPOOL, GAP, CE_HEAD, LAYERNORM, GELU, ATTENTION, TOKENS = range(1, 13)
RULES = {"dp": 0, "v1": 1, "v2": 2}
DTYPES = {"f32": (cdp.CDP_F32, torch.float32, 4), "bf16": (cdp.CDP_BF16, torch.bfloat16, 2)}


def listed():
    return [
        # The smallest model of the benchmark, fp32, with the momentum and weight decay the paper trained with: 20
        # steps whose launches are a few microseconds each.
        dict(name="train_mlp_tiny_f32", kind="train", model="mlp", dtype="f32", stages=4, width=64, inputs=64, classes=10,
             stem=False, N=4, B=8, steps=20, lr=0.05, momentum=0.9, weight_decay=5e-4, rule="v2", dw_group=1),
        # The headline workload: 24 stages of 4096 x 4096, 16 micro-batches of 64, between two looks at the weights.
        dict(name="train_mlp_wide_bf16", kind="train", model="mlp", dtype="bf16", stages=24, width=4096, inputs=4096,
             classes=1000, stem=False, N=16, B=64, steps=20, lr=0.05, momentum=0.0, weight_decay=0.0, rule="v2", dw_group=1),
        # ImageNet-shaped ResNet-50, 8 micro-batches of 32.
        dict(name="train_resnet50_bf16", kind="train", model="resnet50", dtype="bf16", image=224, width=64, classes=1000,
             N=8, B=32, steps=4, lr=0.01, momentum=0.0, weight_decay=0.0, rule="v2", dw_group=1),
        # ViT-B/16-shaped, 8 micro-batches of 32.
        dict(name="train_vit_b16_bf16", kind="train", model="vit", dtype="bf16", stages=12, image=224, patch=16, width=768,
             heads=12, classes=1000, N=8, B=32, steps=4, lr=0.01, momentum=0.0, weight_decay=0.0, rule="v2", dw_group=1),
        # One layer of the smallest model, fp32: what a call costs when there is next to nothing to do.
        dict(name="linear_small_f32", kind="linear", dtype="f32", rows=8, inputs=64, outputs=64),
        # One layer of the headline model.
        dict(name="linear_wide_bf16", kind="linear", dtype="bf16", rows=64, inputs=4096, outputs=4096),
        # A 3x3 convolution of the second group of ResNet-50, 32 images.
        dict(name="conv3x3_bf16", kind="conv", dtype="bf16", B=32, H=28, W=28, cin=128, cout=128, k=3, stride=1, pad=1),
        # The first linear map of a ViT-B MLP on 32 x 196 tokens.
        dict(name="tokens_fc1_bf16", kind="conv", dtype="bf16", B=32, H=1, W=196, cin=768, cout=3072, k=1, stride=1, pad=0),
        # A strided convolution on an odd map in fp32: ResNet-18 on 9 x 9 images.
        dict(name="conv3x3_odd_f32", kind="conv", dtype="f32", B=32, H=9, W=9, cin=64, cout=128, k=3, stride=2, pad=1),
        # The attention core of ViT-B/16 on 32 images.
        dict(name="attention_vit_bf16", kind="attention", dtype="bf16", B=32, T=196, D=768, heads=12),
        # More tokens than a 224 x 224 image gives, fp32.
        dict(name="attention_long_f32", kind="attention", dtype="f32", B=4, T=324, D=192, heads=3),
        # LayerNorm and GELU of a ViT-B block on 32 x 196 tokens.
        dict(name="norm_gelu_bf16", kind="norm_gelu", dtype="bf16", rows=6272, width=768, hidden=3072),
    ]


def _log(rng, lo, hi, step=1):
    """Log-uniform multiple of `step` in [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi // step * step, max(-(-lo // step) * step, round(v / step) * step)))


def draw(rng):
    kind = rng.choice(["train", "linear", "conv", "attention", "norm_gelu"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if kind == "linear":
        return dict(kind=kind, dtype=dtype, rows=rng.randint(4, 128), inputs=_log(rng, 64, 4096, rng.choice([8, 8, 1])),
                    outputs=_log(rng, 64, 4096, rng.choice([8, 8, 1])))
    if kind == "conv":
        what = rng.choice(["k1", "k3", "tokens"])
        if what == "tokens":
            return dict(kind=kind, dtype=dtype, B=_log(rng, 2, 32), H=1, W=rng.randint(16, 256), cin=_log(rng, 64, 1024, 8),
                        cout=_log(rng, 64, 3072, 8), k=1, stride=1, pad=0)
        side = _log(rng, 7, 56)
        stride = rng.choice([1, 1, 1, 2])
        cin = _log(rng, 16, 512 if side <= 28 else 128, 8)
        cout = cin if rng.random() < 0.5 else _log(rng, 16, 512 if side <= 28 else 128, 8)
        return dict(kind=kind, dtype=dtype, B=_log(rng, 2, 32), H=side, W=side, cin=cin, cout=cout, k=3 if what == "k3" else 1,
                    stride=stride, pad=1 if what == "k3" else 0)
    if kind == "attention":
        heads = rng.choice([2, 3, 4, 6, 8, 12])
        return dict(kind=kind, dtype=dtype, B=_log(rng, 2, 32), T=_log(rng, 16, 400), D=heads * rng.choice([16, 32, 40, 64, 64, 80]),
                    heads=heads)
    if kind == "norm_gelu":
        width = _log(rng, 32, 1024, rng.choice([8, 8, 1]))
        return dict(kind=kind, dtype=dtype, rows=_log(rng, 64, 8192), width=width, hidden=4 * width)
    model = rng.choice(["mlp", "mlp", "resnet18", "vit"])
    rule = rng.choice(["v2", "v2", "v1", "dp"])
    c = dict(kind=kind, model=model, dtype=dtype, steps=rng.choice([4, 6, 8]), momentum=rng.choice([0.0, 0.9]), rule=rule, dw_group=1)
    c["weight_decay"] = 5e-4 if c["momentum"] else 0.0
    if model == "mlp":
        S, N = rng.choice([(4, 4), (6, 4), (8, 8), (8, 16), (12, 8)])
        if rule != "dp":
            c["dw_group"] = rng.choice([1, 1, 2])
        c.update(stages=S, N=N, B=rng.randint(4, 64), width=_log(rng, 64, 2048, 8), inputs=_log(rng, 64, 3072, 4), classes=rng.choice([10, 100]),
                 stem=rng.random() < 0.5, lr=0.02)
    elif model == "resnet18":
        c.update(image=rng.randint(8, 32), width=rng.choice([16, 32, 64]), classes=10, N=4, B=rng.randint(4, 32), lr=0.01)
    else:
        heads = rng.choice([2, 3, 4, 6])
        c.update(stages=4, image=rng.choice([32, 48, 64, 96]), patch=8, width=heads * rng.choice([16, 32, 64]), heads=heads, classes=10,
                 N=rng.choice([2, 4]), B=rng.randint(2, 16), lr=0.01)
    if c["momentum"]:
        c["lr"] *= 0.2
    return c


# ---- models: stages as lists of layer descriptors (tensor 0 is the stage input, tensor k + 1 the output of layer k) -----
def _conv_affine(cin, cout, k, stride, pad, src=-1):
    return [Layer(CONV2D, src, (cin, cout, k, stride, pad)), Layer(AFFINE, -1, (cout,))]


def _basic(cin, cout, stride, base):
    ls, short = [], base
    if stride != 1 or cin != cout:
        ls += _conv_affine(cin, cout, 1, stride, 0, base)
        short = base + 2
    ls += _conv_affine(cin, cout, 3, stride, 1, base) + [Layer(RELU, -1, ())] + _conv_affine(cout, cout, 3, 1, 1)
    return ls + [Layer(ADD, -1, (short,)), Layer(RELU, -1, ())]


def _bottleneck(cin, width, stride, base):
    cout, ls, short = 4 * width, [], base
    if stride != 1 or cin != cout:
        ls += _conv_affine(cin, cout, 1, stride, 0, base)
        short = base + 2
    ls += _conv_affine(cin, width, 1, 1, 0, base) + [Layer(RELU, -1, ())]
    ls += _conv_affine(width, width, 3, stride, 1) + [Layer(RELU, -1, ())] + _conv_affine(width, cout, 1, 1, 0)
    return ls + [Layer(ADD, -1, (short,)), Layer(RELU, -1, ())]


def _vit_block(dim, heads, base):
    ls = [Layer(LAYERNORM, base, (dim,))] + _conv_affine(dim, 3 * dim, 1, 1, 0) + [Layer(ATTENTION, -1, (heads,))]
    ls += _conv_affine(dim, dim, 1, 1, 0) + [Layer(ADD, -1, (base,))]
    mid = base + len(ls)
    ls += [Layer(LAYERNORM, -1, (dim,))] + _conv_affine(dim, 4 * dim, 1, 1, 0) + [Layer(GELU, -1, ())]
    return ls + _conv_affine(4 * dim, dim, 1, 1, 0) + [Layer(ADD, -1, (mid,))]


def _model(c):
    """(stages, per-sample input shape, gain of the classifier weights)"""
    if c["model"] == "mlp":
        stages, cin = [], c["inputs"]
        for j in range(c["stages"]):
            st = []
            if j == 0 and c["stem"]:
                st += [Layer(LINEAR, -1, (cin, c["width"])), Layer(RELU, -1, ())]
                cin = c["width"]
            st += [Layer(LINEAR, -1, (cin, c["width"])), Layer(RELU, -1, ())]
            cin = c["width"]
            stages.append(st)
        stages[-1] += [Layer(LINEAR, -1, (cin, c["classes"])), Layer(CE_HEAD, -1, (c["classes"],))]
        return stages, (c["inputs"],), 1.0
    if c["model"] == "vit":
        stages = []
        for j in range(c["stages"]):
            st = _conv_affine(3, c["width"], c["patch"], c["patch"], 0) + [Layer(TOKENS, -1, ())] if j == 0 else []
            stages.append(st + _vit_block(c["width"], c["heads"], len(st)))
        stages[-1] += [Layer(LAYERNORM, -1, (c["width"],)), Layer(GAP, -1, ()), Layer(LINEAR, -1, (c["width"], c["classes"])),
                       Layer(CE_HEAD, -1, (c["classes"],))]
        return stages, (c["image"], c["image"], 3), 0.2
    deep = c["model"] == "resnet50"
    depths, block, grow = ((3, 4, 6, 3), _bottleneck, 4) if deep else ((2, 2, 2, 2), _basic, 1)
    stages, cin = [], c["width"]
    for g, depth in enumerate(depths):
        for b in range(depth):
            st = []
            if not stages and deep:
                st = _conv_affine(3, cin, 7, 2, 3) + [Layer(RELU, -1, ()), Layer(MAXPOOL, -1, (3, 2, 1))]
            elif not stages:
                st = _conv_affine(3, cin, 3, 1, 1) + [Layer(RELU, -1, ())]
            w = c["width"] << g
            st += block(cin, w, 2 if g and not b else 1, len(st))
            cin = grow * w
            stages.append(st)
    stages[-1] += [Layer(GAP, -1, ()), Layer(LINEAR, -1, (cin, c["classes"])), Layer(CE_HEAD, -1, (c["classes"],))]
    return stages, (c["image"], c["image"], 3), 0.05


def _param_shapes(layer):
    p = layer.p
    if layer.kind == LINEAR:
        return [(p[1], p[0]), (p[1],)]
    if layer.kind == CONV2D:
        return [(p[1], p[2], p[2], p[0])]
    if layer.kind in (AFFINE, LAYERNORM):
        return [(p[0],), (p[0],)]
    return []


def _init(stages, head_gain, gen):
    """theta_0 on the GPU: Kaiming-normal weights, zero biases, unit scales (1/4 in front of a residual add)."""
    out = []
    for st in stages:
        ps = []
        for i, l in enumerate(st):
            after = st[i + 1].kind if i + 1 < len(st) else 0
            for k, shape in enumerate(_param_shapes(l)):
                if l.kind in (LINEAR, CONV2D) and k == 0:
                    gain = head_gain if after == CE_HEAD else 1.0
                    ps.append(torch.randn(shape, generator=gen, device="cuda") * (gain * math.sqrt(2.0 / math.prod(shape[1:]))))
                elif l.kind in (AFFINE, LAYERNORM) and k == 0:
                    ps.append(torch.full(shape, 0.25 if after == ADD else 1.0, device="cuda"))
                else:
                    ps.append(torch.zeros(shape, device="cuda"))
        out.append(ps)
    return out


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _train_inputs(c, seed):
    stages, shape, gain = _model(c)
    gen = _gen(seed)
    params = _init(stages, gain, gen)
    rows = c["N"] * c["B"]
    xs = [torch.randn((rows,) + shape, generator=gen, device="cuda") for _ in range(c["steps"])]
    ys = [torch.randint(0, c["classes"], (rows,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(c["steps"])]
    return stages, shape, params, xs, ys


def _layer_inputs(c, seed):
    """Inputs of a single layer, in the case's type; gradients are as small as a mean over a batch makes them."""
    gen, t = _gen(seed), DTYPES[c["dtype"]][1]
    r = lambda *shape, s=1.0: torch.randn(shape, generator=gen, device="cuda").mul_(s).to(t)  # noqa: E731
    if c["kind"] == "linear":
        i, o = c["inputs"], c["outputs"]
        return dict(x=r(c["rows"], i), w=r(o, i, s=math.sqrt(2.0 / i)), dy=r(c["rows"], o, s=0.01))
    if c["kind"] == "conv":
        ho, wo = _conv_out(c)
        fan = c["k"] * c["k"] * c["cin"]
        x = r(c["B"], c["H"], c["W"], c["cin"])
        if c["k"] > 1 or c["H"] > 1:
            x = x.relu_()  # the input of a convolution inside a ResNet comes out of a ReLU
        return dict(x=x, w=r(c["cout"], c["k"], c["k"], c["cin"], s=math.sqrt(2.0 / fan)), dy=r(c["B"], ho, wo, c["cout"], s=0.01))
    if c["kind"] == "attention":
        return dict(qkv=r(c["B"], c["T"], 3 * c["D"], s=1.2), dout=r(c["B"], c["T"], c["D"], s=0.01))
    return dict(x=r(c["rows"], c["width"], s=1.5), h=r(c["rows"], c["hidden"], s=1.2), dy=r(c["rows"], c["width"], s=0.01),
                dh=r(c["rows"], c["hidden"], s=0.01), add=r(c["rows"], c["width"], s=0.01),
                gamma=1 + 0.1 * torch.randn(c["width"], generator=gen, device="cuda"), beta=0.1 * torch.randn(c["width"], generator=gen, device="cuda"))


def _conv_out(c):
    return (c["H"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1


def prepare(case, seed):
    c, t = case, DTYPES[case["dtype"]]
    if c["kind"] == "train":
        stages, shape, params, xs, ys = _train_inputs(c, seed)
        tr = cdp.Trainer(stages, shape, c["N"], c["B"], c["lr"], RULES[c["rule"]], t[0], momentum=c["momentum"],
                         weight_decay=c["weight_decay"], dp_batched=c["rule"] == "dp", dw_group=c["dw_group"])
        for j, ps in enumerate(params):
            cdp.cdp_set_weights(tr.ctx, j, torch.cat([p.reshape(-1) for p in ps]).cpu().numpy())
        return dict(case=c, trainer=tr, xs=xs, ys=ys, done=0)
    s = dict(_layer_inputs(c, seed), case=c)
    new = lambda *shape, d=t[1]: torch.empty(shape, dtype=d, device="cuda")  # noqa: E731
    if c["kind"] == "linear":
        s.update(wt=s["w"].t().contiguous(), y=new(c["rows"], c["outputs"], d=torch.float32), dx=new(c["rows"], c["inputs"], d=torch.float32),
                 dw=new(c["outputs"], c["inputs"], d=torch.float32))
    elif c["kind"] == "conv":
        ho, wo = _conv_out(c)
        ws = 4 * s["w"].numel() * (c["B"] * ho * wo // 512 + 4)
        s.update(wt=s["w"].permute(3, 1, 2, 0).contiguous(), y=new(c["B"], ho, wo, c["cout"]), dx=torch.empty_like(s["x"]),
                 dw=new(*s["w"].shape, d=torch.float32), ws=new(ws, d=torch.uint8))
    elif c["kind"] == "attention":
        tt = c["B"] * c["heads"] * c["T"] * c["T"]
        s.update(P=new(c["B"], c["heads"], c["T"], c["T"]), out=new(c["B"], c["T"], c["D"]), dqkv=torch.empty_like(s["qkv"]),
                 ws=new((4 + t[2]) * tt + 256, d=torch.uint8))
    else:
        w = c["width"]
        s.update(y=torch.empty_like(s["x"]), a=torch.empty_like(s["h"]), da=torch.empty_like(s["h"]), dx=torch.empty_like(s["x"]),
                 dgb=new(2, w, d=torch.float32), ws=new(8 * c["rows"] + 8 * w * -(-c["rows"] // 32) + 256, d=torch.uint8))
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "train":
        tr, first = s["trainer"], s["done"]
        for x, y in zip(s["xs"], s["ys"]):
            tr.step(x, y)
        tr.drain()
        s["done"] += c["steps"]
        return dict(weights=[tr.weights(j) for j in range(tr.S)], losses=np.stack([tr.losses(first + t) for t in range(c["steps"])]))
    dt = DTYPES[c["dtype"]][0]
    p = lambda k: s[k].data_ptr()  # noqa: E731
    st = torch.cuda.current_stream().cuda_stream
    if c["kind"] == "linear":
        m, i, o = c["rows"], c["inputs"], c["outputs"]
        cdp.cdp_k_gemm(dt, 5, 1, 1, p("x"), p("w"), p("y"), m, o, i, i, i, st)
        cdp.cdp_k_gemm(dt, 5, 1, 1, p("dy"), p("wt"), p("dx"), m, i, o, o, o, st)
        cdp.cdp_k_gemm(dt, 0, 0, 0, p("dy"), p("x"), p("dw"), o, i, m, o, i, st)
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"])
    if c["kind"] == "conv":
        g = (c["B"], c["H"], c["W"], c["cin"], c["cout"], c["k"], c["stride"], c["pad"])
        cdp.cdp_k_conv(dt, 0, p("x"), p("w"), p("y"), *g, stream=st)
        cdp.cdp_k_conv(dt, 1, p("dy"), p("wt"), p("dx"), *g, stream=st)
        cdp.cdp_k_conv(dt, 2, p("dy"), p("x"), p("dw"), *g, ws_ptr=p("ws"), ws_bytes=s["ws"].numel(), stream=st)
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"])
    if c["kind"] == "attention":
        g = (p("ws"), s["ws"].numel(), c["B"], c["T"], c["D"], c["heads"], st)
        cdp.cdp_k_attention(dt, 0, p("qkv"), p("P"), 0, p("out"), *g)
        cdp.cdp_k_attention(dt, 1, p("qkv"), p("P"), p("dout"), p("dqkv"), *g)
        return dict(P=s["P"], out=s["out"], dqkv=s["dqkv"])
    r, w, n = c["rows"], c["width"], s["h"].numel()
    cdp.cdp_k_layernorm(dt, 0, p("x"), 0, 0, p("gamma"), p("beta"), p("y"), 0, 0, 0, 0, r, w, st)
    cdp.cdp_k_gelu(dt, 0, p("h"), 0, p("a"), n, st)
    cdp.cdp_k_gelu(dt, 1, p("h"), p("dh"), p("da"), n, st)
    s["dgb"].zero_()
    cdp.cdp_k_layernorm(dt, 1, p("x"), p("dy"), p("add"), p("gamma"), 0, p("dx"), p("dgb"), p("dgb") + 4 * w, p("ws"), s["ws"].numel(), r, w, st)
    return dict(y=s["y"], a=s["a"], da=s["da"], dx=s["dx"], dgb=s["dgb"])


# ---- work ------------------------------------------------------------------------------------------------------------
def _shapes(stages, shape):
    """Per layer of every stage: (layer, input shape, output shape), per sample."""
    out = []
    for st in stages:
        ts, rows = [tuple(shape)], []
        for i, l in enumerate(st):
            a = ts[i if l.src < 0 else l.src]
            if l.kind == LINEAR:
                b = (l.p[1],)
            elif l.kind in (CONV2D, MAXPOOL):
                k, s, q = l.p[-3:]
                b = ((a[0] + 2 * q - k) // s + 1, (a[1] + 2 * q - k) // s + 1, l.p[1] if l.kind == CONV2D else a[2])
            elif l.kind == GAP:
                b = (a[2],)
            elif l.kind == TOKENS:
                b = (1, a[0] * a[1], a[2])
            elif l.kind == ATTENTION:
                b = (1, a[1], a[2] // 3)
            else:
                b = a
            ts.append(b)
            rows.append((l, a, b))
        out.append(rows)
        shape = ts[-1]
    return out


def work(case):
    c, e = case, DTYPES[case["dtype"]][2]
    if c["kind"] == "linear":
        m, i, o = c["rows"], c["inputs"], c["outputs"]
        return dict(flops=6.0 * m * i * o, bytes=float(m * (i + o) * (e + 4) + i * o * (2 * e + 4)))
    if c["kind"] == "conv":
        ho, wo = _conv_out(c)
        x, y, w = c["B"] * c["H"] * c["W"] * c["cin"], c["B"] * ho * wo * c["cout"], c["k"] ** 2 * c["cin"] * c["cout"]
        return dict(flops=6.0 * c["B"] * ho * wo * w, bytes=float(2 * (x + y) * e + w * (2 * e + 4)))
    if c["kind"] == "attention":
        bt, tt = c["B"] * c["T"] * c["D"], c["B"] * c["heads"] * c["T"] ** 2
        # qkv in and dqkv out, out and dout, the probabilities written by one pass and read by the other
        return dict(flops=12.0 * c["B"] * c["T"] ** 2 * c["D"], bytes=float(e * (9 * bt + 2 * bt + 2 * tt)))
    if c["kind"] == "norm_gelu":
        x, h = c["rows"] * c["width"], c["rows"] * c["hidden"]
        return dict(flops=30.0 * (x + h), bytes=float(e * (6 * x + 5 * h)))
    stages, shape, _ = _model(c)
    macs = params = acts = 0
    for st in _shapes(stages, shape):
        for l, a, b in st:
            params += sum(math.prod(s) for s in _param_shapes(l))
            acts += math.prod(b)
            if l.kind == LINEAR:
                macs += l.p[0] * l.p[1]
            elif l.kind == CONV2D:
                macs += math.prod(b[:2]) * l.p[0] * l.p[1] * l.p[2] ** 2
            elif l.kind == ATTENTION:
                macs += 2 * b[1] ** 2 * b[2]
    rows, batches = c["N"] * c["B"], 1 if c["rule"] == "dp" else c["N"]
    # every micro-batch reads every weight in its forward and in its backward (they are a timeline apart), every activation is
    # written once and read once by the backward; a step reads and writes the master weights
    per_step = rows * (4 * math.prod(shape) + 2 * e * acts) + 2 * e * params * batches + 8 * params
    return dict(flops=6.0 * macs * rows * c["steps"], bytes=float(per_step * c["steps"] + 4 * params))


def tolerance(case):
    """Measured against exact(): single layers are 1.7e-3 to 2.7e-3 off in bf16 (the rounding of what is stored) and up to
    1e-6 in fp32, trained weights and losses up to 3.1e-3 in bf16.  In an fp32 training run a few ReLU arguments lie
    within rounding of zero, and a mask that flips there moves the gradients below it."""
    if case["dtype"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": 1e-4} if case["kind"] == "train" else {"rel": 1e-5}


# ---- the same results in 64 bits --------------------------------------------------------------------------------------
def _conv64(x, w, k, stride, pad):
    """NHWC convolution of 64-bit tensors as one matrix product per call; w [cout, k, k, cin]."""
    B, H, W, C = x.shape
    if k == 1:
        cols = x[:, ::stride, ::stride, :]
        return cols @ w.reshape(w.shape[0], -1).t()
    ho, wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    x = F.pad(x, (0, 0, pad, pad, pad, pad))
    cols = torch.cat([x[:, a:a + stride * (ho - 1) + 1:stride, b:b + stride * (wo - 1) + 1:stride, :] for a in range(k) for b in range(k)], dim=3)
    return cols @ w.reshape(w.shape[0], -1).t()


def _attention64(qkv, heads):
    B, T, D3 = qkv.shape
    q, k, v = (z.reshape(B, T, heads, -1).transpose(1, 2) for z in qkv.split(D3 // 3, dim=2))
    P = torch.softmax(q @ k.transpose(2, 3) / math.sqrt(q.shape[-1]), dim=-1)
    return P, (P @ v).transpose(1, 2).reshape(B, T, D3 // 3)


def _stage64(st, ps, x, y):
    ts, it = [x], iter(ps)
    for i, l in enumerate(st):
        a = ts[i if l.src < 0 else l.src]
        if l.kind == LINEAR:
            a = F.linear(a, next(it), next(it))
        elif l.kind == RELU:
            a = a.relu()
        elif l.kind == CONV2D:
            a = _conv64(a, next(it), *l.p[2:])
        elif l.kind == AFFINE:
            a = a * next(it) + next(it)
        elif l.kind == ADD:
            a = a + ts[l.p[0]]
        elif l.kind == MAXPOOL:
            a = F.max_pool2d(a.permute(0, 3, 1, 2), *l.p).permute(0, 2, 3, 1)
        elif l.kind == GAP:
            a = a.mean((1, 2))
        elif l.kind == LAYERNORM:
            a = F.layer_norm(a, (a.shape[-1],), next(it), next(it), 1e-5)
        elif l.kind == GELU:
            a = F.gelu(a)
        elif l.kind == ATTENTION:
            a = _attention64(a[:, 0], l.p[0])[1][:, None]
        elif l.kind == TOKENS:
            a = a.reshape(a.shape[0], 1, -1, a.shape[3])
        else:
            a = F.cross_entropy(a, y.long())
        ts.append(a)
    return ts[-1]


def _train64(c, seed):
    stages, _, params, xs, ys = _train_inputs(c, seed)
    S, N, B = len(stages), c["N"], c["B"]
    cur = [[p.double() for p in ps] for ps in params]
    old, vel = cur, [[torch.zeros_like(p) for p in ps] for ps in cur]
    delay = 0 if c["rule"] == "dp" else 2 * S // N
    losses = torch.zeros(c["steps"], N, dtype=torch.float64)
    for t, (x, y) in enumerate(zip(xs, ys)):
        total = [[torch.zeros_like(p) for p in ps] for ps in cur]
        for i in range(N):
            # a stage's parameters of this step are there once the last micro-batch of the step before has updated them
            fresh = [c["rule"] == "dp" or (c["rule"] == "v2" and delay * (N - 1 - i) <= 2 * j) for j in range(S)]
            point = [[p.detach().requires_grad_() for p in (cur if fresh[j] else old)[j]] for j in range(S)]
            a, rows = x[i * B:(i + 1) * B].double(), y[i * B:(i + 1) * B]
            for j in range(S):
                a = _stage64(stages[j], point[j], a, rows)
            losses[t, i] = a.item()
            a.backward()
            for tot, ps in zip(total, point):
                for u, p in zip(tot, ps):
                    u += p.grad
            del a, point
        new = []
        for j in range(S):
            row = []
            for p, v, g in zip(cur[j], vel[j], total[j]):
                v.mul_(c["momentum"]).add_(g / N + c["weight_decay"] * p)
                row.append(p - c["lr"] * v)
            new.append(row)
        old, cur = cur, new
    return dict(weights=[torch.cat([p.reshape(-1) for p in ps]).cpu().numpy() for ps in cur], losses=losses.numpy())


def exact(case, seed):
    c = case
    if c["kind"] == "train":
        return _train64(c, seed)
    s = {k: v.double() for k, v in _layer_inputs(c, seed).items()}
    if c["kind"] == "linear":
        return dict(y=s["x"] @ s["w"].t(), dx=s["dy"] @ s["w"], dw=s["dy"].t() @ s["x"])
    if c["kind"] == "conv":
        x, w = s["x"].requires_grad_(), s["w"].requires_grad_()
        y = _conv64(x, w, c["k"], c["stride"], c["pad"])
        dx, dw = torch.autograd.grad(y, (x, w), s["dy"])
        return dict(y=y.detach(), dx=dx, dw=dw)
    if c["kind"] == "attention":
        qkv = s["qkv"].requires_grad_()
        P, out = _attention64(qkv, c["heads"])
        return dict(P=P.detach(), out=out.detach(), dqkv=torch.autograd.grad(out, qkv, s["dout"])[0])
    x, h, g, b = (s[k].requires_grad_() for k in ("x", "h", "gamma", "beta"))
    y, a = F.layer_norm(x, (c["width"],), g, b, 1e-5), F.gelu(h)
    dx, dg, db = torch.autograd.grad(y, (x, g, b), s["dy"])
    return dict(y=y.detach(), a=a.detach(), da=torch.autograd.grad(a, h, s["dh"])[0], dx=dx + s["add"], dgb=torch.stack([dg, db]))
