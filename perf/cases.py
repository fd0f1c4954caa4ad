"""The work that is timed on this framework: one pipeline stage's mini-batch step
(forward of every micro-batch, backward with recomputation, update fused with
the next predictions), forwards alone, and the flat update and prediction
passes, through the public entry points.

A stage case names a small network and its sizes; its layers, parameters and
inputs follow from the case and the seed.  Sizes come from the stages that the
repository trains and benchmarks: VGG-16 on 32 x 32 images (micro-batch 32),
ResNet-101 and Inception-V3 on 224 x 224 images (micro-batch 100), the
Inception-A stage on 35 x 35 maps (micro-batch 32) and the small MLP.

First moments start at zero and second moments as the paper draws them
(1e-4 U(0, 1)), so that after the update m / (1 - beta1) is the gradient
accumulated over the mini-batch: a step's outputs hold every gradient.  In a
whole stage of many ReLU layers the bf16 gradients are not unique (a change of
rounding in one layer flips masks in all that follow, several per cent of the
gradient's norm), so those cases return outputs, losses and updated weights."""
import math

import torch
import torch.nn.functional as F

import paper_1911_04610_amd as xp

LR, BETA1, BETA2, EPS, BN_EPS = 1e-3, 0.9, 0.999, 1e-8, 1e-5
RULES = {"sgd": xp.RULE_MOMENTUM_SGD, "rmsprop": xp.RULE_RMSPROP}


# ---------------------------------------------------------------- networks
def _layers(case):
    """The case's layer list."""
    out = []

    def add(**kw):
        out.append(kw)
        return len(out) - 1

    def conv(x, cin, cout, k, kw=None, stride=1, pad="same", bias=False):
        return add(kind="conv", inputs=[x], cin=cin, cout=cout, k=k, kw=kw or k, stride=stride, pad=pad, bias=bias)

    def relu(x):
        return add(kind="relu", inputs=[x])

    def bn(x, c):
        return add(kind="bn", inputs=[x], cin=c, cout=c)

    def cbr(x, cin, cout, k, **kw):
        return relu(bn(conv(x, cin, cout, k, **kw), cout))

    net, cin, cout = case["net"], case.get("cin", 0), case.get("cout", 0)
    if net == "mlp":
        h = relu(add(kind="linear", inputs=[-1], cin=cin, cout=cout, bias=True))
        z = add(kind="linear", inputs=[h], cin=cout, cout=case["classes"], bias=True)
        add(kind="softmax_ce", inputs=[z], classes=case["classes"])
    elif net == "conv":  # one convolution with its BN and ReLU
        cbr(-1, cin, cout, case["k"], kw=case.get("kw"), stride=case.get("stride", 1), pad=case.get("pad", "same"))
    elif net == "vgg":  # the end of a VGG-16 block: two convolutions with bias and ReLU, and the pool
        x = relu(conv(-1, cin, cout, 3, bias=True))
        x = relu(conv(x, cout, cout, 3, bias=True))
        add(kind="maxpool2", inputs=[x])
    elif net == "stem":  # ResNet-101's first layers
        add(kind="maxpool3s2", inputs=[cbr(-1, cin, cout, 7, stride=2)])
    elif net in ("projection", "identity"):  # bottleneck blocks; cin = cout for the identity shortcut
        x, c = -1, cin
        for _ in range(case.get("blocks", 1)):
            mid, stride = case["mid"], case.get("stride", 1)
            y = cbr(cbr(x, c, mid, 1), mid, mid, 3, stride=stride)
            short = x
            if net == "projection":
                short = bn(conv(x, c, cout, 1, stride=stride), cout)
            y = bn(conv(y, mid, cout, 1), cout)
            x, c = relu(add(kind="add", inputs=[y, short])), cout
    elif net == "inception_a":  # Inception-A modules, then pooling, classifier and loss
        x, c = -1, cin
        for _ in range(case["modules"]):
            b1 = cbr(x, c, 64, 1)
            b2 = cbr(cbr(x, c, 48, 1), 48, 64, 5)
            b3 = cbr(cbr(cbr(x, c, 64, 1), 64, 96, 3), 96, 96, 3)
            b4 = cbr(add(kind="avgpool3", inputs=[x]), c, 32, 1)
            x, c = add(kind="concat", inputs=[b1, b2, b3, b4]), 256
        z = add(kind="linear", inputs=[add(kind="gap", inputs=[x])], cin=c, cout=case["classes"], bias=True)
        add(kind="softmax_ce", inputs=[z], classes=case["classes"])
    elif net == "head":  # global average pooling, classifier, loss
        z = add(kind="linear", inputs=[add(kind="gap", inputs=[-1])], cin=cin, cout=case["classes"], bias=True)
        add(kind="softmax_ce", inputs=[z], classes=case["classes"])
    else:
        raise ValueError(net)
    return out


def _in_shape(case):
    return (case["cin"],) if case["net"] == "mlp" else (case["h"], case["w"], case["cin"])


def _shapes(case):
    """[n, H, W, C] of every layer's output and, at -1, of the input."""
    s = _in_shape(case)
    shapes = {-1: (case["micro"],) + ((1, 1) + s if len(s) == 1 else s)}
    for i, L in enumerate(_layers(case)):
        n, h, w, c = shapes[L["inputs"][0]]
        kind, same = L["kind"], L.get("pad", "same") == "same"
        if kind == "conv":
            st, ph, pw = L["stride"], L["k"] // 2 * same, L["kw"] // 2 * same
            h, w, c = (h + 2 * ph - L["k"]) // st + 1, (w + 2 * pw - L["kw"]) // st + 1, L["cout"]
        elif kind == "linear":
            c = L["cout"]
        elif kind == "maxpool2":
            h, w = h // 2, w // 2
        elif kind == "maxpool3s2":
            h, w = (h - 1) // 2 + 1, (w - 1) // 2 + 1
        elif kind == "gap":
            h, w = 1, 1
        elif kind == "concat":
            c = sum(shapes[j][3] for j in L["inputs"])
        shapes[i] = (n, h, w, c)
    return shapes


def _params(layers):
    """(layer index, role, shape) of every parameter tensor, in buffer order."""
    out = []
    for i, L in enumerate(layers):
        if L["kind"] in ("conv", "linear"):
            out.append((i, "weight", (L["cout"], L["k"], L["kw"], L["cin"]) if L["kind"] == "conv" else (L["cout"], L["cin"])))
            if L["bias"]:
                out.append((i, "bias", (L["cout"],)))
        elif L["kind"] == "bn":
            out += [(i, "gamma", (L["cout"],)), (i, "beta", (L["cout"],))]
    return out


def _deep(case):
    """Whole stages, whose bf16 gradients are not unique."""
    return case["dtype"] == "bf16" and case["net"] in ("identity", "inception_a")


def _loss(case):
    return case["net"] in ("mlp", "head", "inception_a")


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest step: launches and their latency (the repository's MLP, four micro-batches)
        dict(name="mlp_step_f32", net="mlp", mode="step", dtype="f32", micro=32, T=4, cin=256, cout=256, classes=10, s_fwd=2, s_bwd=2),
        # the update at the mini-batch boundary on a ResNet-101 stage's parameters, with both next predictions
        dict(name="update_adam", net="flat", op="adam", n=10_734_217, s_fwd=1, s_bwd=1),
        # the end of VGG-16's fourth block: few rows, deep reductions
        dict(name="vgg_4x4", net="vgg", mode="step", dtype="bf16", micro=32, T=4, cin=512, cout=512, h=4, w=4, s_fwd=1, s_bwd=1),
        # Inception-A's 3 x 3 branch convolution, the headline stage's most frequent kernel
        dict(name="conv3x3_35", net="conv", mode="step", dtype="bf16", micro=32, T=4, cin=64, cout=96, k=3, h=35, w=35, s_fwd=1, s_bwd=1),
        # an asymmetric convolution of Inception-C on its odd 12 x 12 maps
        dict(name="conv7x1_12", net="conv", mode="step", dtype="bf16", micro=100, T=2, cin=160, cout=192, k=7, kw=1, h=12, w=12, s_fwd=1, s_bwd=1),
        # a forward pass alone, few samples of ResNet-101's last group (evaluation of a stage)
        dict(name="forward_7x7", net="conv", mode="forward", dtype="bf16", micro=8, T=1, cin=512, cout=512, k=3, h=7, w=7, s_fwd=0, s_bwd=0),
        # ResNet-101's stem: 3 channels, stride 2, the largest maps
        dict(name="stem_224", net="stem", mode="step", dtype="bf16", micro=100, T=1, cin=3, cout=64, h=224, w=224, s_fwd=1, s_bwd=1),
        # the first block of ResNet-101's first group: the largest activations, bound by memory
        dict(name="block_56", net="projection", mode="step", dtype="bf16", micro=100, T=1, cin=64, mid=64, cout=256, h=56, w=56, s_fwd=1, s_bwd=1),
        # the first block of its third group: strided, wide products
        dict(name="block_28_s2", net="projection", mode="step", dtype="bf16", micro=100, T=1, cin=512, mid=256, cout=1024, stride=2, h=28, w=28, s_fwd=1, s_bwd=1),
        # two of the 22 blocks that fill the network's middle stages, forwards beside backwards
        dict(name="blocks_14", net="identity", mode="step", overlap=True, dtype="bf16", micro=100, T=2, blocks=2, cin=1024, mid=256, cout=1024, h=14, w=14, s_fwd=1, s_bwd=1),
        # a middle bottleneck in the 32-bit storage format
        dict(name="block_16_f32", net="identity", mode="step", dtype="f32", micro=32, T=1, cin=512, mid=128, cout=512, h=16, w=16, s_fwd=1, s_bwd=1),
        # the headline benchmark's whole step: the Inception-A stage, forwards beside backwards
        dict(name="inception_a_step", net="inception_a", mode="step", overlap=True, dtype="bf16", micro=32, T=4, modules=3, cin=256, classes=200, h=35, w=35, s_fwd=1, s_bwd=1),
    ]


def draw(rng):
    """One more case of the same ranges: any layer of the networks above, micro-batches
    of 1 to 128, square, oblong and odd maps, channel counts on and off the usual multiples."""
    def logint(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    def channels(a, b):
        c = logint(a, b)
        return c if rng.random() < 0.15 else max(8, (c + 4) // 8 * 8) if rng.random() < 0.4 else max(16, (c + 16) // 32 * 32)

    while True:
        kind = rng.choice(["flat", "mlp", "conv", "conv", "conv", "conv", "forward", "vgg", "stem", "projection", "identity", "head", "f32"])
        s_fwd, s_bwd = rng.choice([(1, 1), (2, 1), (1, 2), (0, 0)])
        if kind == "flat":
            return dict(net="flat", op=rng.choice(["adam", "predict", "sgd", "rmsprop"]), n=logint(10_000, 60_000_000), s_fwd=s_fwd, s_bwd=s_bwd)
        case = dict(net=kind, mode="step", dtype="bf16", micro=logint(1, 128), T=rng.choice([1, 1, 2, 4]), s_fwd=s_fwd, s_bwd=s_bwd)
        if kind == "mlp":
            case.update(dtype=rng.choice(["f32", "bf16"]), cin=channels(64, 2048), cout=channels(64, 2048), classes=rng.choice([10, 100, 200]))
            return case
        h = logint(4, 70)
        case.update(h=h, w=h if rng.random() < 0.6 else max(4, h + rng.randint(-5, 5)))
        if kind in ("conv", "forward", "f32"):
            k, kw = rng.choice([(1, 1), (1, 1), (3, 3), (3, 3), (5, 5), (1, 7), (7, 1), (1, 3)])
            case.update(net="conv", cin=channels(32, 1024), cout=channels(32, 1024), k=k, kw=kw,
                        stride=rng.choice([1, 1, 1, 2]), pad="valid" if h > k and case["w"] > kw and rng.random() < 0.15 else "same")
            if kind == "forward":
                case.update(mode="forward", T=1)
            if kind == "f32":
                case.update(dtype="f32", cin=channels(32, 256), cout=channels(32, 256))
        elif kind == "vgg":
            case.update(cin=rng.choice([3, 64, 128, 256, 512]), cout=rng.choice([64, 128, 256, 512]), h=h // 2 * 2, w=case["w"] // 2 * 2)
        elif kind == "stem":
            case.update(cin=3, cout=rng.choice([32, 64]), h=rng.randint(32, 224), w=rng.randint(32, 224))
        elif kind == "projection":
            mid = rng.choice([64, 96, 128, 256])
            case.update(cin=channels(64, 1024), mid=mid, cout=4 * mid, stride=rng.choice([1, 2]))
        elif kind == "identity":
            mid = rng.choice([64, 128, 256])
            case.update(cin=4 * mid, mid=mid, cout=4 * mid, blocks=rng.choice([1, 2]), overlap=rng.random() < 0.5)
        elif kind == "head":
            case.update(cin=channels(64, 2048), classes=rng.choice([10, 100, 200]), h=logint(3, 35))
            case["w"] = case["h"]
        # batch statistics over a handful of values, or gradients of a handful of
        # rows, have no stable digits to compare
        shapes = _shapes(case)
        if case["net"] != "head" and min(n * a * b for i, (n, a, b, c) in shapes.items() if i < len(shapes) - 2) < 64:
            continue
        # no more than the largest listed step, nor than the largest listed activations
        w = work(case)
        acts = sum(n * a * b * c for n, a, b, c in shapes.values()) * (4 if case["dtype"] == "f32" else 2)
        if w["flops"] <= (2e10 if case["dtype"] == "f32" else 6e11) and acts <= 8e8 and w["bytes"] <= 8e8:
            return case


# ---------------------------------------------------------------- inputs
def _draw_inputs(case, seed):
    """The case's parameters, moments and data: tensors on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=g, device="cuda") * std

    if case["net"] == "flat":
        n = case["n"]
        return dict(W=normal(n, std=0.02), m=normal(n, std=1e-3), v=normal(n, std=1e-6).abs(), G=normal(n, std=1e-3),
                    buf=normal(n, std=1e-3) if case["op"] in RULES else None,
                    sq=normal(n, std=1e-6).abs() if case["op"] == "rmsprop" else None)
    layers, shapes = _layers(case), _shapes(case)
    tdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    params, v = [], []
    for _, role, shape in _params(layers):
        if role == "weight":  # Kaiming uniform
            a = math.sqrt(6.0 / math.prod(shape[1:]))
            params.append((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * a)
        else:
            params.append(torch.full(shape, 1.0 if role == "gamma" else 0.0, device="cuda"))
        v.append(1e-4 * torch.rand(shape, generator=g, device="cuda"))
    T, last = case["T"], shapes[len(layers) - 1]
    # images and the first layer's inputs are normal, a later layer's input is the ReLU output before it
    x = [normal(*shapes[-1]) for _ in range(T)]
    if case["net"] != "mlp" and case["cin"] > 3:
        x = [t.relu_() for t in x]
    if case["net"] == "mlp":
        x = [t.reshape(case["micro"], case["cin"]) for t in x]
    dy = labels = None
    if _loss(case):
        labels = [torch.randint(0, case["classes"], (case["micro"],), generator=g, device="cuda", dtype=torch.int32) for _ in range(T)]
    elif case["mode"] == "step":
        dy = [normal(*last, std=1e-2).to(tdt) for _ in range(T)]
    return dict(params=params, v=v, x=[t.to(tdt) for t in x], dy=dy, labels=labels)


def prepare(case, seed):
    d = _draw_inputs(case, seed)
    hyper = xp.Hyper(lr=LR, beta1=BETA1, beta2=BETA2, eps=EPS)
    if case["net"] == "flat":
        d.update(case=case, hyper=hyper, t=100, pred_fwd=torch.empty_like(d["W"]), pred_bwd=torch.empty_like(d["W"]))
        if case["op"] in RULES:
            d["rule"] = xp.Rule(rule=RULES[case["op"]], lr=LR, momentum=0.9, weight_decay=5e-4, alpha=0.99, eps=1e-8)
        return d
    dtype, tdt = (xp.BF16, torch.bfloat16) if case["dtype"] == "bf16" else (xp.F32, torch.float32)
    st = xp.Stage(_layers(case), case["micro"], case["T"], _in_shape(case), dtype)
    for (off, cnt), p, v in zip(st.layout, d["params"], d["v"]):
        st.W[off:off + cnt] = p.reshape(-1)
        st.v[off:off + cnt] = v.reshape(-1)
    T = case["T"]
    y = [torch.empty(st.out_shape, dtype=tdt, device="cuda") for _ in range(T)]
    loss = torch.zeros(T, device="cuda") if _loss(case) else None
    # the first stage has no input gradient to send
    dx = [torch.empty_like(x) for x in d["x"]] if case["net"] not in ("stem", "mlp") and case["mode"] == "step" and case["cin"] > 3 else None
    state = dict(case=case, hyper=hyper, t=0, stage=st, x=d["x"], dy=d["dy"], labels=d["labels"], y=y, loss=loss,
                 losses=None if loss is None else [loss[i:i + 1] for i in range(T)], dx=dx, fwd=None)
    st.xpipe_predict_weights(xp.FWD, case["s_fwd"], hyper, 0)
    st.xpipe_predict_weights(xp.BWD, case["s_bwd"], hyper, 0)
    if case.get("overlap"):
        state["fwd"] = st.xpipe_stage_set_fwd_stream(True)
    return state


# ---------------------------------------------------------------- one pass
def _run_flat(s):
    op, W, m, v, G = s["case"]["op"], s["W"], s["m"], s["v"], s["G"]
    pf, pb, sf, sb = s["pred_fwd"], s["pred_bwd"], s["case"]["s_fwd"], s["case"]["s_bwd"]
    if op == "predict":
        xp.xpipe_predict_flat(W, m, v, pf, None, sf, s["hyper"], s["t"])
        return {"pred_fwd": pf}
    if op == "adam":
        xp.xpipe_adam_flat(W, m, v, G, s["hyper"], s["t"], True, pf, sf, pb, sb)
        out = {}
    else:
        xp.xpipe_rule_flat(W, s["buf"], s["sq"], m, v, G, s["rule"], s["hyper"], s["t"], True, pf, sf, pb, sb)
        out = {"buf": s["buf"]} if op == "sgd" else {"buf": s["buf"], "sq": s["sq"]}
    return dict(out, W=W, m=m, v=v, G=G, pred_fwd=pf, pred_bwd=pb)


def run(s):
    case = s["case"]
    if case["net"] == "flat":
        return _run_flat(s)
    st, x, y, labels, losses = s["stage"], s["x"], s["y"], s["labels"], s["losses"]
    T = case["T"]

    def forward(i):
        st.xpipe_stage_fwd(x[i], y[i], labels[i] if labels else None, losses[i] if losses else None)

    if case["mode"] == "forward":
        forward(0)
        return {"y": y}
    dy, dx = s["dy"], s["dx"]

    def backward(i):
        st.xpipe_stage_bwd(x[i], dy[i] if dy else None, labels[i] if labels else None, dx[i] if dx else None)

    if s["fwd"] is not None:
        s["fwd"].wait_stream(torch.cuda.current_stream())
    for i in range(T):  # the steady state's order: a forward, then a backward
        forward(i)
        backward(i)
    st.xpipe_adam_step(s["hyper"], s["t"], case["s_fwd"], case["s_bwd"], emit_pred=True)
    if s["fwd"] is not None:
        torch.cuda.current_stream().wait_stream(s["fwd"])
    s["t"] += 1
    if _deep(case):
        return {"y": y, "loss": s["loss"], "W": st.W}
    return {"y": y, "loss": s["loss"], "dx": dx, "W": st.W, "m": st.m, "v": st.v, "pred_fwd": st.w_pred_fwd, "pred_bwd": st.w_pred_bwd}


# ---------------------------------------------------------------- what it cannot do without
def work(case):
    if case["net"] == "flat":
        # predict: W, m, v in, one prediction out; updates: the state in and out, G in and zeroed, two predictions out
        words = {"predict": 4, "adam": 10, "sgd": 12, "rmsprop": 14}[case["op"]]
        return {"bytes": 4.0 * words * case["n"], "flops": 10.0 * case["n"]}
    layers, shapes = _layers(case), _shapes(case)
    elem = 2 if case["dtype"] == "bf16" else 4
    step, T = case["mode"] == "step", case["T"]
    size = {i: math.prod(s) for i, s in shapes.items()}
    has_dx = case["net"] not in ("stem", "mlp") and case["cin"] > 3
    flops, params = 0.0, sum(math.prod(s) for _, _, s in _params(layers))
    for i, L in enumerate(layers):
        if L["kind"] in ("conv", "linear"):
            one = 2.0 * size[i] * L["cin"] * (L["k"] * L["kw"] if L["kind"] == "conv" else 1)
            # forward; recomputed forward, weight gradient and input gradient
            flops += one * ((3 + (L["inputs"] != [-1] or has_dx)) if step else 1)
    act = size[-1] + size[len(layers) - 1 - _loss(case)]  # x and y
    if step:
        act += size[-1] * has_dx + (0 if _loss(case) else size[len(layers) - 1])  # dx and dy
    # the update reads W, m, v and writes them and both predictions; a forward reads the prediction
    return {"bytes": float(T * act * elem + params * 4 * (8 if step else 1)), "flops": T * flops}


def tolerance(case):
    """32-bit results are rounded once from 64-bit sums (3e-8 to 1e-7 off the exact ones).

    bf16: an output is 2.6e-3 off the exact one, one rounding of a stored value,
    and four times that is stated for single layers.  With the fp32 sums in another
    order alone, a single layer moves by 2e-5 to 7e-4 (a value that rounds the other
    way is up to 1.4e-2 off), the gradients of a block of three ReLU layers by 1e-3
    (maps of 56 x 56) to 7.6e-3 (0.56 at a flipped mask), and the outputs of whole
    stages by 2e-3 to 3.3e-3."""
    if case["net"] == "flat" or case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    if case["net"] == "projection":
        return {"rel": 3e-2, "max": 0.99}
    return {"rel": 1.3e-2 if _deep(case) else 1e-2, "max": 0.4}


# ---------------------------------------------------------------- the same in 64 bits
def _conv64(x, w, stride, ph, pw):
    """x [n, H, W, C], w [N, R, S, C]: one product per filter tap."""
    N, R, S, C = w.shape
    x = F.pad(x, (0, 0, pw, pw, ph, ph))
    ho, wo = (x.shape[1] - R) // stride + 1, (x.shape[2] - S) // stride + 1
    y = 0
    for r in range(R):
        for q in range(S):
            t = x[:, r:r + stride * (ho - 1) + 1:stride, q:q + stride * (wo - 1) + 1:stride].reshape(-1, C)
            y = y + t @ w[:, r, q].t()
    return y.reshape(x.shape[0], ho, wo, N)


def _pool64(x, k, stride, pad):
    y = F.max_pool2d(x.permute(0, 3, 1, 2), k, stride, pad)
    return y.permute(0, 2, 3, 1)


def _forward64(layers, params, x, labels, minibatch):
    """The stage's output and, with labels, its share of the mini-batch loss."""
    val, it, loss = {-1: x}, iter(params), None
    for i, L in enumerate(layers):
        a, kind = val[L["inputs"][0]], L["kind"]
        if kind == "conv":
            same = L["pad"] == "same"
            a = _conv64(a, next(it), L["stride"], L["k"] // 2 * same, L["kw"] // 2 * same)
            a = a + next(it) if L["bias"] else a
        elif kind == "linear":
            a = a @ next(it).t() + next(it)
        elif kind == "bn":
            mean = a.mean((0, 1, 2))
            var = (a - mean).square().mean((0, 1, 2))
            a = (a - mean) / (var + BN_EPS).sqrt() * next(it) + next(it)
        elif kind == "relu":
            a = a.relu()
        elif kind == "add":
            a = a + val[L["inputs"][1]]
        elif kind == "maxpool2":
            a = _pool64(a, 2, 2, 0)
        elif kind == "maxpool3s2":
            a = _pool64(a, 3, 2, 1)
        elif kind == "avgpool3":
            b = F.pad(a, (0, 0, 1, 1, 1, 1))
            n, h, w, _ = a.shape
            a = sum(b[:, r:r + h, q:q + w] for r in range(3) for q in range(3)) / 9
        elif kind == "gap":
            a = a.mean((1, 2), keepdim=True)
        elif kind == "concat":
            a = torch.cat([val[j] for j in L["inputs"]], 3)
        elif kind == "softmax_ce":
            loss = F.cross_entropy(a.reshape(a.shape[0], -1), labels.long(), reduction="sum") / minibatch
        val[i] = a
    return a, loss


def _adam64(W, m, v, g, t):
    """State after update t + 1, and its prediction's direction."""
    m, v = BETA1 * m + (1 - BETA1) * g, BETA2 * v + (1 - BETA2) * g * g
    mh, vh = m / (1 - BETA1 ** (t + 1)), v / (1 - BETA2 ** (t + 1))
    return W - LR * mh / (vh.sqrt() + EPS), m, v, mh / (vh + EPS).sqrt()


def _exact_flat(case, d):
    W, m, v, G = (d[k].double() for k in ("W", "m", "v", "G"))
    if case["op"] == "predict":
        t = 100
        way = m / (1 - BETA1 ** t) / (v / (1 - BETA2 ** t) + EPS).sqrt()
        return {"pred_fwd": W - case["s_fwd"] * LR * way}
    if case["op"] == "adam":
        W, m, v, way = _adam64(W, m, v, G, 100)
        out = {}
    else:
        g, buf = G + 5e-4 * W, d["buf"].double()
        _, m, v, way = _adam64(W, m, v, g, 100)
        if case["op"] == "sgd":
            buf = 0.9 * buf + g
            out = {"buf": buf}
        else:
            sq = 0.99 * d["sq"].double() + 0.01 * g * g
            buf = 0.9 * buf + g / (sq.sqrt() + 1e-8)
            out = {"buf": buf, "sq": sq}
        W = W - LR * buf
    return dict(out, W=W, m=m, v=v, G=torch.zeros_like(W), pred_fwd=W - case["s_fwd"] * LR * way, pred_bwd=W - case["s_bwd"] * LR * way)


def exact(case, seed):
    d = _draw_inputs(case, seed)
    if case["net"] == "flat":
        return _exact_flat(case, d)
    layers, T = _layers(case), case["T"]
    roles = _params(layers)
    step = case["mode"] == "step" and not _deep(case)
    # the products' weight operands are the prediction rounded to the storage format
    params = [(p.to(torch.bfloat16) if case["dtype"] == "bf16" and role == "weight" else p).double().requires_grad_(step)
              for p, (_, role, _) in zip(d["params"], roles)]
    ys, dxs, losses = [], [], []
    for i in range(T):
        x = d["x"][i].double().reshape(_shapes(case)[-1])
        if step:
            x.requires_grad_(True)
        with torch.set_grad_enabled(step):
            y, loss = _forward64(layers, params, x, d["labels"][i] if d["labels"] else None, T * case["micro"])
            if step:
                if loss is not None:
                    loss.backward()
                else:
                    (y * d["dy"][i].double()).sum().backward()
                dxs.append(x.grad.reshape(d["x"][i].shape))
        ys.append(y.detach())
        losses.append(loss.detach() if loss is not None else None)
        del x, y, loss
    loss = torch.stack(losses) if losses[0] is not None else None
    if case["mode"] == "forward":
        return {"y": ys}
    if not step:
        return {"y": ys, "loss": loss, "W": None}
    has_dx = case["net"] not in ("stem", "mlp") and case["cin"] > 3
    flat = {k: [] for k in ("W", "m", "v", "pred_fwd", "pred_bwd")}
    for p, v, q in zip(d["params"], d["v"], params):
        W = p.double().reshape(-1)
        W, m, v, way = _adam64(W, torch.zeros_like(W), v.double().reshape(-1), q.grad.reshape(-1), 0)
        for k, t in (("W", W), ("m", m), ("v", v), ("pred_fwd", W - case["s_fwd"] * LR * way), ("pred_bwd", W - case["s_bwd"] * LR * way)):
            flat[k].append(F.pad(t, (0, -t.numel() % 64)))
    return dict({k: torch.cat(t) for k, t in flat.items()}, y=ys, loss=loss, dx=dxs if has_dx else None)
