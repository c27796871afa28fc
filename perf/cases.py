"""The work whose time counts: training steps and forward passes of single layers, and the policy-gradient loss.

Every case is what one layer of a Caffe-style training program asks of the library per iteration, through the
Python binding: the forward pass, the data gradient (a first layer needs none) and the parameter gradients, on
blobs, a descriptor and a workspace that such a program allocates once.  Sizes are the repository's own layer
shapes (``paper_1810_02272_amd/workloads.py``); ``draw`` spreads them over the ranges those shapes span.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

import paper_1810_02272_amd as lib

DEV = "cuda"


def _conv(name, n, c, h, w, k, kh, kw, sh=1, sw=1, ph=0, pw=0, dh=1, dw=1, group=1, step="train", dtype="f32",
          x="normal", wstd=0.01, dystd=0.1):
    """step: "train" (forward, data gradient, filter + bias gradients), "first" (a first layer's step: no data
    gradient) or "forward" (inference).  wstd 0: Xavier-uniform weights."""
    return dict(name=name, kind="conv", n=n, c=c, h=h, w=w, k=k, kh=kh, kw=kw, sh=sh, sw=sw, ph=ph, pw=pw, dh=dh,
                dw=dw, group=group, step=step, dtype=dtype, x=x, wstd=wstd, dystd=dystd)


def listed():
    return [
        # first layer of a digit network, 28x28x1 images, batch 64: the smallest training step
        _conv("digits_first", 64, 1, 28, 28, 20, 5, 5, step="first", x="uniform01", wstd=0.0, dystd=1.0),
        # its second layer: small image, whole step
        _conv("digits_second", 64, 20, 12, 12, 50, 5, 5, x="uniform01", wstd=0.0, dystd=1.0),
        # second layer of a small-image (32x32x3) network, batch 100
        _conv("small_image_second", 100, 32, 16, 16, 32, 5, 5, ph=2, pw=2, dystd=1.0),
        # the three convolution layers of a large-image network, batch 128
        _conv("large_image_first", 128, 3, 227, 227, 96, 11, 11, 4, 4, step="first"),
        _conv("large_image_grouped", 128, 96, 27, 27, 256, 5, 5, ph=2, pw=2, group=2),
        _conv("large_image_third", 128, 256, 13, 13, 384, 3, 3, ph=1, pw=1),
        # one image through a trained layer: latency of a forward pass
        _conv("one_image_forward", 1, 96, 27, 27, 256, 5, 5, ph=2, pw=2, group=2, step="forward"),
        # nothing a multiple of anything: strided layer with ragged channels and a non-square image
        _conv("ragged_strided", 37, 45, 51, 67, 77, 3, 5, 2, 1, 1, 2),
        # depthwise layer of a mobile-style network
        _conv("depthwise", 64, 128, 56, 56, 128, 3, 3, ph=1, pw=1, group=128, wstd=0.0, dystd=1.0),
        # the double base type on an ordinary layer
        _conv("third_doubles", 32, 256, 13, 13, 384, 3, 3, ph=1, pw=1, dtype="f64"),
        # the widest fully connected layer, ReLU fused, batch 128
        dict(name="inner_product", kind="ip", m=128, k=9216, o=4096, relu=1),
        # both policy-gradient models on a batch of finished episodes
        dict(name="policy_gradient", kind="pg", episodes=65536, min_len=8, max_len=500, actions=6, gamma=0.99),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    r = rng.random()
    if r < 0.12:
        return dict(kind="ip", m=_log_int(rng, 1, 200), k=_log_int(rng, 64, 9216), o=_log_int(rng, 10, 4096),
                    relu=rng.randrange(2))
    if r < 0.2:
        hi = _log_int(rng, 20, 500)
        return dict(kind="pg", episodes=_log_int(rng, 64, 60000), min_len=rng.randint(1, 8), max_len=hi,
                    actions=rng.randint(2, 18), gamma=rng.choice((0.9, 0.99)))
    while True:
        kh = rng.choice((1, 3, 3, 3, 3, 4, 5, 5, 7, 8, 11))
        kw = kh if rng.random() < 0.8 else rng.choice((1, 3, 5))
        sh = rng.choice((1, 1, 1, 2, 4) if kh >= 7 else (1, 1, 1, 1, 2))
        sw = sh if rng.random() < 0.9 else rng.choice((1, 2))
        dil = 2 if kh in (3, 5) and sh == 1 and rng.random() < 0.1 else 1
        step = rng.choice(("train", "train", "train", "train", "forward"))
        c = _log_int(rng, 1, 384)
        if c <= 4 and step == "train" and rng.random() < 0.5:
            step = "first"
        k = _log_int(rng, 8, 384)
        group = 1
        g = rng.random()
        if g < 0.12:
            group = c = k = max(c, 8)
        elif g < 0.25:
            group = rng.choice((2, 2, 4))
            c, k = max(1, c // group) * group, max(1, k // group) * group
        h = _log_int(rng, 7, 227)
        case = _conv("", _log_int(rng, 1, 128), c, h, h if rng.random() < 0.6 else max(7, h + rng.randint(-h // 3, h // 3)),
                     k, kh, kw, sh, sw, rng.randint(0, dil * (kh - 1) // 2), rng.randint(0, dil * (kw - 1) // 2), dil,
                     dil, group, step, "f64" if rng.random() < 0.15 else "f32", rng.choice(("normal", "uniform01")),
                     rng.choice((0.0, 0.01)), rng.choice((0.1, 1.0)))
        del case["name"]
        oh, ow = _out(case)
        if oh < 1 or ow < 1:
            continue
        # what the widest tiles would make of it, so that a drawn case stays under the largest listed one
        padded = 2.0 * case["n"] * oh * ow * group * (-(-(k // group) // 16) * 16) * (-(-(c // group) * kh * kw // 16) * 16)
        heavy = case["dtype"] == "f64"
        if group == c == k and c > 1:
            padded = 40.0 * case["n"] * k * oh * ow * kh * kw
        if padded > (6e9 if heavy else 3e10):
            continue
        if max(case["n"] * c * h * case["w"], case["n"] * k * oh * ow) > (1 << 24 if heavy else 1 << 25):
            continue
        return case


def _out(case):
    return ((case["h"] + 2 * case["ph"] - case["dh"] * (case["kh"] - 1) - 1) // case["sh"] + 1,
            (case["w"] + 2 * case["pw"] - case["dw"] * (case["kw"] - 1) - 1) // case["sw"] + 1)


def _normal(shape, gen, std, dtype=torch.float32):
    return torch.empty(shape, device=DEV, dtype=dtype).normal_(0.0, std, generator=gen)


def _uniform(shape, gen, lo, hi, dtype=torch.float32):
    return torch.empty(shape, device=DEV, dtype=dtype).uniform_(lo, hi, generator=gen)


def _conv_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    oh, ow = _out(case)
    xs = (case["n"], case["c"], case["h"], case["w"])
    ws = (case["k"], case["c"] // case["group"], case["kh"], case["kw"])
    x = _uniform(xs, gen, 0.0, 1.0, dt) if case["x"] == "uniform01" else _normal(xs, gen, 1.0, dt)
    a = math.sqrt(3.0 / (ws[1] * ws[2] * ws[3]))
    w = _normal(ws, gen, case["wstd"], dt) if case["wstd"] else _uniform(ws, gen, -a, a, dt)
    b = _uniform((case["k"],), gen, -0.1, 0.1, dt)
    dy = _normal((case["n"], case["k"], oh, ow), gen, case["dystd"], dt) if case["step"] != "forward" else None
    return x, w, b, dy


def _ip_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    m, k, o = case["m"], case["k"], case["o"]
    x = _normal((m, k), gen, 1.0)
    w = _normal((o, k), gen, 0.01)
    b = _uniform((o,), gen, -0.1, 0.1)
    dy = _normal((m, o), gen, 0.1)
    # The ReLU mask is a yes/no decision on a float: it is taken on stored activations (zero on half of the
    # places, as after a ReLU), so that a rounding of the forward sums near zero cannot flip a gradient.
    act = _normal((m, o), gen, 1.0).clamp_(min=0.0)
    return x, w, b, dy, act


def _pg_inputs(case, seed):
    cpu = torch.Generator().manual_seed(seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    # lengths spread evenly over their range, in an order of the seed's: batches of one size
    span = case["max_len"] - case["min_len"] + 1
    lengths = case["min_len"] + torch.randperm(case["episodes"], generator=cpu) * span // case["episodes"]
    offsets = torch.zeros(case["episodes"] + 1, dtype=torch.int64)
    offsets[1:] = torch.cumsum(lengths, 0)
    steps = int(offsets[-1])
    reward = torch.ones(steps, device=DEV)  # pole balancing: 1 per step, 0 on the step that ends an episode
    reward[(offsets[1:] - 1).to(DEV)] = 0.0
    aprob = _uniform((steps,), gen, 0.01, 0.99)
    random = _uniform((steps,), gen, 0.0, 1.0)
    logits = _normal((steps, case["actions"]), gen, 2.0)
    action = torch.randint(0, case["actions"], (steps,), generator=gen, device=DEV, dtype=torch.int32)
    return offsets.to(torch.int32).to(DEV), reward, aprob, random, logits, action, lengths


def prepare(case, seed):
    if case["kind"] == "conv":
        x, w, b, dy = _conv_inputs(case, seed)
        f64 = case["dtype"] == "f64"
        d = lib.conv_desc_create(lib.ConvParams(
            n=case["n"], c=case["c"], h=case["h"], w=case["w"], num_output=case["k"], kernel_h=case["kh"],
            kernel_w=case["kw"], stride_h=case["sh"], stride_w=case["sw"], pad_h=case["ph"], pad_w=case["pw"],
            dilation_h=case["dh"], dilation_w=case["dw"], group=case["group"]))
        size = lib.conv_desc_workspace_bytes_f64(d) if f64 else lib.conv_desc_workspace_bytes(d)
        s = dict(kind="conv64" if f64 else "conv", step=case["step"], d=d, x=x, w=w, b=b, dy=dy,
                 y=torch.empty(lib.conv_desc_output_shape(d), device=DEV, dtype=x.dtype),
                 ws=torch.empty((size + 7) // 8, device=DEV, dtype=torch.float64))
        if case["step"] != "forward":
            s["dw"], s["db"] = torch.empty_like(w), torch.empty_like(b)
        if case["step"] == "train":
            s["dx"] = torch.empty_like(x)
        return s
    if case["kind"] == "ip":
        x, w, b, dy, act = _ip_inputs(case, seed)
        d = lib.ip_desc_create(lib.IpParams(m=case["m"], k=case["k"], num_output=case["o"], relu=case["relu"]))
        return dict(kind="ip", d=d, x=x, w=w, b=b, dy=dy, act=act, y=torch.empty_like(dy), dz=torch.empty_like(dy),
                    dx=torch.empty_like(x), dw=torch.empty_like(w), db=torch.empty_like(b),
                    ws=torch.empty((lib.ip_desc_workspace_bytes(d) + 3) // 4, device=DEV))
    offsets, reward, aprob, random, logits, action, _ = _pg_inputs(case, seed)
    one = torch.empty_like(reward)
    return dict(kind="pg", offsets=offsets, reward=reward, aprob=aprob, random=random, logits=logits, action=action,
                gamma=case["gamma"], sampled=torch.empty_like(action), r=one, dlogps=torch.empty_like(one),
                sdiff=torch.empty_like(one), probs=torch.empty_like(logits), diff=torch.empty_like(logits))


def run(s):
    if s["kind"] == "conv":
        d, ws = s["d"], s["ws"]
        lib.conv_forward(d, s["x"], s["w"], s["b"], s["y"], ws)
        if s["step"] == "forward":
            return [s["y"]]
        out = [s["y"], s["dw"], s["db"]]
        if s["step"] == "train":
            lib.conv_backward_data(d, s["w"], s["dy"], s["dx"], ws)
            out.append(s["dx"])
        lib.conv_backward_filter_bias(d, s["x"], s["dy"], s["dw"], s["db"], 0.0, ws)
        return out
    if s["kind"] == "conv64":
        d, ws = s["d"], s["ws"]
        lib.conv_forward_f64(d, s["x"], s["w"], s["b"], s["y"], ws)
        if s["step"] == "forward":
            return [s["y"]]
        out = [s["y"], s["dw"], s["db"]]
        if s["step"] == "train":
            lib.conv_backward_data_f64(d, s["w"], s["dy"], s["dx"], ws)
            out.append(s["dx"])
        lib.conv_backward_filter_f64(d, s["x"], s["dy"], s["dw"], 0.0, ws)
        lib.conv_backward_bias_f64(d, s["dy"], s["db"], 0.0, ws)
        return out
    if s["kind"] == "ip":
        d, ws = s["d"], s["ws"]
        lib.ip_forward(d, s["x"], s["w"], s["b"], s["y"], ws)
        lib.ip_relu_backward(d, s["act"], s["dy"], s["dz"])
        lib.ip_backward_filter(d, s["x"], s["dz"], s["dw"], 0.0, ws)
        lib.ip_backward_bias(d, s["dz"], s["db"], 0.0, ws)
        lib.ip_backward_data(d, s["w"], s["dz"], s["dx"], ws)
        return [s["y"], s["dz"], s["dw"], s["db"], s["dx"]]
    lib.pg_sigmoid_sample_action(s["aprob"], s["random"], s["sampled"])
    lib.pg_discount_rewards(s["reward"], s["offsets"], s["gamma"], s["r"])
    lib.pg_sigmoid_bottom_diff(s["aprob"], s["sampled"], s["r"], s["dlogps"], s["sdiff"])
    lib.pg_softmax_bottom_diff(s["logits"], s["action"], s["r"], s["probs"], s["diff"])
    return [s["sampled"], s["r"], s["dlogps"], s["sdiff"], s["probs"], s["diff"]]


def work(case):
    if case["kind"] == "conv":
        oh, ow = _out(case)
        item = 8 if case["dtype"] == "f64" else 4
        x = case["n"] * case["c"] * case["h"] * case["w"]
        y = case["n"] * case["k"] * oh * ow
        w = case["k"] * (case["c"] // case["group"]) * case["kh"] * case["kw"]
        flops = 2.0 * y * (case["c"] // case["group"]) * case["kh"] * case["kw"]
        if case["step"] == "forward":
            return {"bytes": item * (x + w + case["k"] + y), "flops": flops}
        if case["step"] == "first":  # x, w, b, dy in; y, dw, db out
            return {"bytes": item * (x + 2 * w + 2 * case["k"] + 2 * y), "flops": 2 * flops}
        return {"bytes": item * (2 * x + 2 * w + 2 * case["k"] + 2 * y), "flops": 3 * flops}
    if case["kind"] == "ip":
        m, k, o = case["m"], case["k"], case["o"]
        # x, w, b, dy, act in; y, dz, dx, dw, db out
        return {"bytes": 4 * (2 * m * k + 2 * o * k + 2 * o + 4 * m * o), "flops": 6.0 * m * k * o}
    steps = case["episodes"] * (case["min_len"] + case["max_len"]) / 2
    # in: reward, aprob, random, action, logits; out: sampled, R, dlogps, diff, probs, diff (softmax)
    return {"bytes": 4 * steps * (4 + 4 + 3 * case["actions"]), "flops": steps * (12 + 8.0 * case["actions"])}


def tolerance(case):
    # about four times the largest error against 64 bits that any output of the listed and drawn cases shows
    if case["kind"] == "conv" and case["dtype"] == "f64":
        return {"rel": 2e-14}
    if case["kind"] == "pg":
        return {"rel": 2e-6, "differ": 0.0}
    return {"rel": 5e-6}


def _exact_conv(case, seed):
    x, w, b, dy = _conv_inputs(case, seed)
    n, c, k, g, kh, kw = case["n"], case["c"], case["k"], case["group"], case["kh"], case["kw"]
    oh, ow = _out(case)
    how = dict(kernel_size=(kh, kw), dilation=(case["dh"], case["dw"]), padding=(case["ph"], case["pw"]),
               stride=(case["sh"], case["sw"]))
    w2 = w.double().view(g, k // g, -1)
    y = torch.empty((n, k, oh, ow), device=DEV, dtype=torch.float64)
    dx = torch.empty((n, c, case["h"], case["w"]), device=DEV, dtype=torch.float64)
    dw = torch.zeros_like(w2)
    per = max(1, min(n, int(1.5e8 // max(1, c * kh * kw * oh * ow))))  # images at a time
    for i in range(0, n, per):
        m = min(per, n - i)
        cols = F.unfold(x[i:i + m].double(), **how).view(m, g, -1, oh * ow)
        for q in range(g):
            y[i:i + m].view(m, g, k // g, oh * ow)[:, q] = torch.matmul(w2[q], cols[:, q])
        if dy is None:
            continue
        top = dy[i:i + m].double().view(m, g, k // g, oh * ow)
        for q in range(g):
            dw[q] += torch.bmm(top[:, q].contiguous(), cols[:, q].transpose(1, 2).contiguous()).sum(0)
        if case["step"] == "train":
            back = torch.empty_like(cols)
            for q in range(g):
                back[:, q] = torch.matmul(w2[q].t().contiguous(), top[:, q])
            dx[i:i + m] = F.fold(back.view(m, -1, oh * ow), output_size=(case["h"], case["w"]), **how)
    y += b.double().view(1, k, 1, 1)
    if dy is None:
        return [y]
    out = [y, dw.view(w.shape), dy.double().sum((0, 2, 3))]
    return out + [dx] if case["step"] == "train" else out


def exact(case, seed):
    if case["kind"] == "conv":
        return _exact_conv(case, seed)
    if case["kind"] == "ip":
        x, w, b, dy, act = (t.double() for t in _ip_inputs(case, seed))
        y = x @ w.t() + b
        dz = torch.where(act > 0, dy, torch.zeros_like(dy)) if case["relu"] else dy
        return [y.clamp(min=0.0) if case["relu"] else y, dz, dz.t() @ x, dz.sum(0), dz @ w]
    offsets, reward, aprob, random, logits, action, lengths = _pg_inputs(case, seed)
    gamma = float(torch.tensor(case["gamma"], dtype=torch.float32))  # the entry point takes a 32-bit float
    start, lengths = offsets[:-1].long(), lengths.to(DEV)
    r = torch.zeros(reward.numel(), device=DEV, dtype=torch.float64)
    later = torch.zeros(case["episodes"], device=DEV, dtype=torch.float64)
    for back in range(1, int(lengths.max()) + 1):  # all episodes one step further from their ends
        live = lengths >= back
        at = (start + lengths - back)[live]
        later[live] = reward[at].double() + gamma * later[live]
        r[at] = later[live]
    sampled = (random >= aprob).int()
    dlogps = torch.where(sampled == 0, 1.0 - aprob.double(), -aprob.double())
    probs = torch.softmax(logits.double(), 1)
    diff = probs.clone()
    diff[torch.arange(diff.shape[0], device=DEV), action.long()] -= 1.0
    return [None, r, dlogps, -dlogps * r, probs, diff * r[:, None]]
