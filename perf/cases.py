"""The work a user of this library has it do, as a list of timed cases: convolution layers (forward, kernel gradient,
input gradient), pooling, fully connected layers, the explicit unroll and its adjoint, and one whole training pass, each
through the public calls of `paper_1501_07338_amd`.  `listed()` takes its sizes from the five benchmark networks of
`workloads.py` (and the mini-batch sweep around them); `draw()` gives more of the same kinds over the ranges they span.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_1501_07338_amd import vcnn
from paper_1501_07338_amd import workloads as wl
from paper_1501_07338_amd.net import TrainStep

DEV = "cuda:0"
MAX_FLOPS = 1.6e11   # of a drawn convolution, all passes together: below the largest listed layer by a wide margin
MAX_PATCH = 1.2e8    # entries of a drawn layer's patch matrix
MAX_ELEMS = 3.0e7    # elements of any one tensor of a drawn case


def _conv(name, n, c, h, w, k, r, s, ph=0, pw=0, relu=True, dtype="f32", dx=True, bwd=True):
    return dict(name=name, kind="conv", n=n, c=c, h=h, w=w, k=k, r=r, s=s, ph=ph, pw=pw, relu=relu, dtype=dtype, dx=dx,
                bwd=bwd)


def listed():
    return [
        # the smallest call: a first layer on eight digit images (cfg1), all launch latency; a network's first layer
        # has no input gradient
        _conv("first_conv", 8, 1, 28, 28, 6, 5, 5, dx=False),
        # the whole digit network (cfg2) at the mini-batch of the experiments: twenty short launches in a chain
        dict(name="digits_step", kind="net", net="cfg2", batch=128),
        # its larger fully connected layer, forward and backward
        dict(name="digits_fc", kind="fc", batch=128, i=800, o=500, relu=True, dtype="f32"),
        # the middle layer of the colour recognition network (cfg3): many small images, 'same' padding
        _conv("colour_conv2", 128, 32, 15, 15, 32, 5, 5, 2, 2),
        # first layer of the denoising network (cfg4): one channel, large planes, bandwidth and latency
        _conv("denoise_conv1", 64, 1, 64, 64, 64, 9, 9, 4, 4, dx=False),
        # its main layer: 64 -> 32 maps, 'same' padding
        _conv("denoise_conv2", 64, 64, 64, 64, 32, 5, 5, 2, 2),
        # the deconvolution network (cfg5): a long one-dimensional kernel over an odd number of maps, valid
        _conv("deconv_separable", 16, 38, 64, 184, 38, 1, 121),
        # its dominant layer, 0.38 TFLOP a pass: the largest call
        _conv("deconv_dense", 16, 38, 64, 64, 512, 16, 16),
        # the same layer in the bfloat16 variant
        _conv("deconv_dense_bf16", 16, 38, 64, 64, 512, 16, 16, dtype="bf16"),
        # its 1 x 1 layer: a plain product over 49 x 49 planes (rows on odd boundaries)
        _conv("deconv_pointwise", 16, 512, 49, 49, 512, 1, 1),
        # overlapping max pooling of the colour network's first maps, forward and backward, at a large mini-batch
        dict(name="colour_pool", kind="pool", n=1024, c=32, h=32, w=32, win=3, stride=2, mode="max", dtype="f32"),
        # phi_c and phi_c^{-1} as calls of their own, on the denoising network's main layer at a quarter of its batch
        dict(name="unroll", kind="unroll", n=16, c=64, h=64, w=64, r=5, s=5, ph=2, pw=2, dtype="f32"),
    ]


# ---- drawn cases ----------------------------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_conv(rng):
    while True:
        shape = rng.choice(["square", "square", "square", "large", "pointwise", "tall", "wide"])
        if shape == "square":
            r = s = rng.choice([3, 4, 5, 5, 7, 9])
        elif shape == "large":
            r, s = rng.randint(8, 16), rng.randint(8, 16)
        elif shape == "pointwise":
            r = s = 1
        else:
            r, s = _log_int(rng, 8, 121), 1
            if shape == "wide":
                r, s = s, r
        h, w = _log_int(rng, 7, 184), _log_int(rng, 7, 184)
        if rng.random() < 0.5:
            w = h
        ph = pw = 0
        if r % 2 == 1 and s % 2 == 1 and rng.random() < 0.4:
            ph, pw = r // 2, s // 2
        n = _log_int(rng, 1, 400)
        c = 1 if rng.random() < 0.15 else _log_int(rng, 3, 512)
        k = 1 if rng.random() < 0.1 else _log_int(rng, 6, 512)
        oh, ow = h + 2 * ph - r + 1, w + 2 * pw - s + 1
        if oh < 1 or ow < 1:
            continue
        flops = 3 * 2.0 * k * c * r * s * n * oh * ow
        if not 1e6 <= flops <= MAX_FLOPS or c * r * s * n * oh * ow > MAX_PATCH:
            continue
        if max(n * c * h * w, n * k * oh * ow) > MAX_ELEMS or k * c * r * s > MAX_ELEMS:
            continue
        case = _conv("", n, c, h, w, k, r, s, ph, pw, relu=rng.random() < 0.6,
                     dtype="bf16" if rng.random() < 0.3 else "f32", dx=c > 1, bwd=rng.random() < 0.75)
        del case["name"]
        return case


def draw(rng):
    kind = rng.choice(["conv"] * 8 + ["fc", "fc", "pool", "pool", "unroll", "net"])
    dtype = "bf16" if rng.random() < 0.3 else "f32"
    if kind == "conv":
        return _draw_conv(rng)
    if kind == "fc":
        return dict(kind="fc", batch=_log_int(rng, 1, 512), i=_log_int(rng, 64, 4096), o=_log_int(rng, 10, 1024),
                    relu=rng.random() < 0.5, dtype=dtype)
    if kind == "net":
        return dict(kind="net", net=rng.choice(["cfg2", "cfg3"]), batch=_log_int(rng, 1, 300))
    while True:
        n, c, h, w = _log_int(rng, 1, 1024), _log_int(rng, 3, 128), _log_int(rng, 7, 128), _log_int(rng, 7, 128)
        if kind == "pool":
            win, stride = rng.choice([(2, 2), (3, 2), (3, 3), (2, 1)])
            if 1e4 <= n * c * h * w <= MAX_ELEMS:
                return dict(kind="pool", n=n, c=c, h=h, w=w, win=win, stride=stride,
                            mode="avg" if rng.random() < 0.25 else "max", dtype=dtype)
        else:
            r, s = rng.randint(1, 9), rng.randint(1, 9)
            ph, pw = (r // 2, s // 2) if r % 2 and s % 2 and rng.random() < 0.5 else (0, 0)
            oh, ow = h + 2 * ph - r + 1, w + 2 * pw - s + 1
            if oh >= 1 and ow >= 1 and 1e4 <= c * r * s * n * oh * ow <= MAX_PATCH:
                return dict(kind="unroll", n=n, c=c, h=h, w=w, r=r, s=s, ph=ph, pw=pw, dtype=dtype)


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _dt(case):
    return (vcnn.BF16, torch.bfloat16) if case["dtype"] == "bf16" else (vcnn.F32, torch.float32)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * seed + 17)
    return g


def _normal(gen, shape, scale=1.0):
    return torch.randn(shape, generator=gen, device=DEV) * scale


def _layer_input(gen, shape):
    """What reaches a layer: an image scaled to [0, 1] (at most 4 channels), else the rectified maps of the layer below."""
    if len(shape) == 4 and shape[1] <= 4:
        return torch.rand(shape, generator=gen, device=DEV)
    return _normal(gen, shape).clamp_(min=0)


def _gradient(gen, shape, masked):
    """The gradient that comes down from the layer above, zero where this layer's rectifier was off."""
    g = _normal(gen, shape, 1e-2)
    return g * (torch.rand(shape, generator=gen, device=DEV) < 0.5) if masked else g


def _conv_tensors(case, seed):
    gen = _gen(seed)
    dt = _dt(case)[1]
    n, c, h, w, k, r, s = (case[q] for q in "nchwkrs")
    oh, ow = h + 2 * case["ph"] - r + 1, w + 2 * case["pw"] - s + 1
    x = _layer_input(gen, (n, c, h, w)).to(dt)
    wgt = _normal(gen, (k, c, r, s), math.sqrt(2.0 / (c * r * s))).to(dt)
    bias = _normal(gen, (k,), 0.1)
    dy = _gradient(gen, (n, k, oh, ow), case["relu"]).to(dt) if case["bwd"] else None
    return x, wgt, bias, dy


def _fc_tensors(case, seed):
    gen = _gen(seed)
    dt = _dt(case)[1]
    b, i, o = case["batch"], case["i"], case["o"]
    return (_layer_input(gen, (b, i)).to(dt), _normal(gen, (o, i), math.sqrt(2.0 / i)).to(dt), _normal(gen, (o,), 0.1),
            _gradient(gen, (b, o), case["relu"]).to(dt))


def _pool_tensors(case, seed):
    gen = _gen(seed)
    dt = _dt(case)[1]
    oh, ow = (case["h"] - case["win"]) // case["stride"] + 1, (case["w"] - case["win"]) // case["stride"] + 1
    return (_layer_input(gen, (case["n"], case["c"], case["h"], case["w"])).to(dt),
            _gradient(gen, (case["n"], case["c"], oh, ow), False).to(dt))


def _unroll_tensors(case, seed):
    gen = _gen(seed)
    n, c, h, w, r, s = (case[q] for q in "nchwrs")
    oh, ow = h + 2 * case["ph"] - r + 1, w + 2 * case["pw"] - s + 1
    return _layer_input(gen, (n, c, h, w)).to(_dt(case)[1]), _normal(gen, (c * r * s, n * oh * ow), 1e-2)


def _net_tensors(case, seed):
    """The network's own seeded generators, moved to another stream of numbers by the seed."""
    net = wl.make_net(case["net"], case["batch"])
    rng = np.random.Generator(np.random.Philox(key=77_000_000 + seed))
    inputs, params = wl.make_inputs(net), wl.make_params(net)
    inputs["x"] = (rng.random(inputs["x"].shape) if case["net"] == "cfg2"
                   else rng.standard_normal(inputs["x"].shape)).astype(np.float32)
    inputs["labels"] = rng.integers(0, net.classes, size=inputs["labels"].shape).astype(np.int32)
    params = [None if p is None else
              ((rng.standard_normal(p[0].shape) * math.sqrt(2.0 / np.prod(p[0].shape[1:]))).astype(np.float32), p[1])
              for p in params]
    return net, inputs, params


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _desc(case):
    return vcnn.conv_desc(case["n"], case["c"], case["h"], case["w"], case.get("k", 1), case["r"], case["s"], case["ph"],
                          case["pw"], dtype=_dt(case)[0],
                          act=vcnn.ACT_RELU if case.get("relu") else vcnn.ACT_NONE)


def prepare(case, seed):
    if case["kind"] == "net":
        net, inputs, params = _net_tensors(case, seed)
        return dict(case=case, step=TrainStep(net, params, inputs, device=DEV))
    vdt, dt = _dt(case)
    if case["kind"] == "conv":
        x, wgt, bias, dy = _conv_tensors(case, seed)
        d = _desc(case)
        oh, ow = vcnn.conv_out_shape(d)
        passes = [vcnn.PASS_FWD] + ([vcnn.PASS_BWD_FILTER, vcnn.PASS_BWD_DATA] if case["bwd"] else [])
        ws = max(vcnn.conv_workspace_bytes(d, p) for p in passes)
        st = dict(case=case, d=d, x=x, w=wgt, bias=bias, dy=dy, y=_empty((case["n"], case["k"], oh, ow), dt),
                  ws=_empty(max(ws, 256), torch.uint8))
        if case["bwd"]:
            st.update(dw=_empty(wgt.shape, torch.float32), db=_empty(bias.shape, torch.float32))
            if case["dx"]:
                st["dx"] = _empty(x.shape, dt)
        return st
    if case["kind"] == "fc":
        x, wgt, bias, dy = _fc_tensors(case, seed)
        return dict(case=case, vdt=vdt, x=x, w=wgt, bias=bias, dy=dy, y=_empty(dy.shape, dt),
                    dw=_empty(wgt.shape, torch.float32), db=_empty(bias.shape, torch.float32), dx=_empty(x.shape, dt))
    if case["kind"] == "pool":
        x, dy = _pool_tensors(case, seed)
        d = vcnn.pool_desc(case["n"], case["c"], case["h"], case["w"], case["win"], case["win"], case["stride"],
                           case["stride"], dtype=vdt, mode=vcnn.POOL_MAX if case["mode"] == "max" else vcnn.POOL_AVG)
        return dict(case=case, d=d, x=x, dy=dy, y=_empty(dy.shape, dt),
                    argmax=_empty(dy.shape, torch.int32) if case["mode"] == "max" else None, dx=_empty(x.shape, dt))
    x, col_in = _unroll_tensors(case, seed)
    return dict(case=case, d=_desc(case), x=x, col=_empty(col_in.shape, dt), col_in=col_in, dx=_empty(x.shape, dt))


# ---- one pass -------------------------------------------------------------------------------------------------------
def run(st):
    case = st["case"]
    if case["kind"] == "conv":
        d, x, w, dy, ws = st["d"], st["x"], st["w"], st["dy"], st["ws"]
        vcnn.conv_fwd(d, x, w, st["bias"], st["y"], ws)
        out = dict(y=st["y"])
        if case["bwd"]:
            if case["dx"]:
                vcnn.conv_bwd_data(d, w, dy, st["dx"], ws)
                out["dx"] = st["dx"]
            vcnn.conv_bwd_filter(d, x, dy, st["dw"], st["db"], ws)
            out.update(dw=st["dw"], db=st["db"])
        return out
    if case["kind"] == "fc":
        b, i, o = case["batch"], case["i"], case["o"]
        act = vcnn.ACT_RELU if case["relu"] else vcnn.ACT_NONE
        vcnn.fc_fwd(st["vdt"], b, i, o, act, st["x"], st["w"], st["bias"], st["y"])
        vcnn.fc_bwd(st["vdt"], b, i, o, st["x"], st["w"], st["dy"], st["dw"], st["db"], st["dx"])
        return {q: st[q] for q in ("y", "dw", "db", "dx")}
    if case["kind"] == "pool":
        vcnn.pool_fwd(st["d"], st["x"], st["y"], st["argmax"])
        vcnn.pool_bwd(st["d"], st["dy"], st["argmax"], st["dx"])
        out = dict(y=st["y"], dx=st["dx"])
        if st["argmax"] is not None:
            out["argmax"] = st["argmax"]
        return out
    if case["kind"] == "unroll":
        vcnn.im2col(st["d"], st["x"], st["col"])
        vcnn.col2im(st["d"], st["col_in"], st["dx"])
        return dict(col=st["col"], dx=st["dx"])
    ts = st["step"]  # forward, cost and backward; the weights stay, so every pass starts from the same state
    ts.forward()
    ts.cost()
    ts.backward()
    return dict(logits=ts.acts[-1], loss=ts.loss, grads=[t for g in ts.grads if g is not None for t in g])


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def work(case):
    e = 2 if case.get("dtype") == "bf16" else 4
    if case["kind"] == "conv":
        n, c, h, w, k, r, s = (case[q] for q in "nchwkrs")
        oh, ow = h + 2 * case["ph"] - r + 1, w + 2 * case["pw"] - s + 1
        x, wt, y = n * c * h * w, k * c * r * s, n * k * oh * ow
        one = 2.0 * wt * n * oh * ow
        nbytes, flops = e * (x + wt + y) + 4 * k, one
        if case["bwd"]:
            nbytes += e * y + 4 * wt + 4 * k + (e * x if case["dx"] else 0)
            flops += one * (2 if case["dx"] else 1)
        return dict(bytes=nbytes, flops=flops)
    if case["kind"] == "fc":
        b, i, o = case["batch"], case["i"], case["o"]
        return dict(bytes=e * (2 * b * i + i * o + 2 * b * o) + 4 * (i * o + 2 * o), flops=6.0 * b * i * o)
    if case["kind"] == "pool":
        oh, ow = (case["h"] - case["win"]) // case["stride"] + 1, (case["w"] - case["win"]) // case["stride"] + 1
        src, dst = case["n"] * case["c"] * case["h"] * case["w"], case["n"] * case["c"] * oh * ow
        index = 8 * dst if case["mode"] == "max" else 0
        return dict(bytes=2 * e * (src + dst) + index, flops=float(dst * case["win"] ** 2))
    if case["kind"] == "unroll":
        n, c, h, w, r, s = (case[q] for q in "nchwrs")
        oh, ow = h + 2 * case["ph"] - r + 1, w + 2 * case["pw"] - s + 1
        src, col = n * c * h * w, c * r * s * n * oh * ow
        return dict(bytes=2 * e * src + (e + 4) * col, flops=float(col))
    net = wl.make_net(case["net"], case["batch"])
    nbytes = flops = 0
    for li, layer in enumerate(net.layers):
        src, dst = float(np.prod(net.in_shape(li))), float(np.prod(net.shapes[li]))
        back = 1 if li > 0 else 0  # no gradient of the network's input
        if isinstance(layer, wl.Pool):
            nbytes += 4 * (src + 2 * dst + dst + back * src)
            flops += dst * layer.win ** 2
            continue
        wt = layer.cout * net.in_shape(li)[1] * layer.kh * layer.kw if isinstance(layer, wl.Conv) else \
            layer.out * src / net.batch
        per = 2.0 * wt * (dst / layer.cout if isinstance(layer, wl.Conv) else net.batch)
        nbytes += 4 * (src + wt + dst + dst + wt + back * src)
        flops += per * (2 + back)
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["kind"] == "unroll":  # phi_c copies; phi_c^{-1} adds at most 81 floats (and rounds once where dx is bfloat16)
        return {"rel": 4e-3} if case["dtype"] == "bf16" else {"rel": 1e-6}
    if case["kind"] == "pool":    # copies, or sums of at most nine values
        return {"rel": 4e-3, "differ": 0.0} if case["dtype"] == "bf16" else {"rel": 1e-6, "differ": 0.0}
    if case["kind"] == "net":
        # the logits agree to 1e-6; but a rectifier or a pooling window whose decision lies within rounding of a tie may
        # fall either way, which moves one whole term of a gradient's sum over some 1e5
        return {"rel": 4e-3}
    if case["dtype"] == "bf16":   # one rounding of the result to eight bits
        return {"rel": 1e-2}
    # sums of up to 1e5 floats: 1.2e-6 (largest element 2.5e-5) from the sums in 64 bits, and so twice that between two
    # orders of the sum
    return {"rel": 6e-6, "max": 1e-4}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------
def _exact_conv(case, seed):
    x, wgt, bias, dy = (None if t is None else t.double() for t in _conv_tensors(case, seed))
    n, c, h, w, k, r, s = (case[q] for q in "nchwkrs")
    pad = (case["ph"], case["pw"])
    oh, ow = h + 2 * pad[0] - r + 1, w + 2 * pad[1] - s + 1
    w2 = wgt.reshape(k, -1)
    y = torch.empty((n, k, oh, ow), dtype=torch.float64, device=DEV)
    out = dict(y=y)
    if case["bwd"]:
        dw = torch.zeros_like(w2)
        if case["dx"]:
            out["dx"] = torch.empty_like(x)
    step = max(1, int(1.5e8) // (c * r * s * oh * ow))
    for a in range(0, n, step):
        b = min(n, a + step)
        cols = F.unfold(x[a:b], (r, s), padding=pad).permute(1, 0, 2).reshape(c * r * s, -1).contiguous()
        yy = torch.mm(w2, cols) + bias[:, None]
        y[a:b] = (yy.clamp(min=0) if case["relu"] else yy).reshape(k, b - a, oh, ow).permute(1, 0, 2, 3)
        if case["bwd"]:
            d2 = dy[a:b].permute(1, 0, 2, 3).reshape(k, -1).contiguous()
            dw += torch.mm(d2, cols.t().contiguous())
            if case["dx"]:
                dcol = torch.mm(w2.t().contiguous(), d2).reshape(c * r * s, b - a, oh * ow).permute(1, 0, 2).contiguous()
                out["dx"][a:b] = F.fold(dcol, (h, w), (r, s), padding=pad)
    if case["bwd"]:
        out.update(dw=dw.reshape(wgt.shape), db=dy.sum(dim=(0, 2, 3)))
    return out


def _exact_net(case, seed):
    net, inputs, params = _net_tensors(case, seed)
    a, leaves = torch.from_numpy(inputs["x"]).double(), []
    for layer, p in zip(net.layers, params):
        if isinstance(layer, wl.Pool):
            a = F.max_pool2d(a, layer.win, layer.stride)
            continue
        w, b = (torch.from_numpy(t).double().requires_grad_() for t in p)
        leaves += [w, b]
        if isinstance(layer, wl.Conv):
            a = F.conv2d(a, w, b, padding=(layer.pad_h, layer.pad_w))
        else:
            a = F.linear(a.reshape(a.shape[0], -1), w, b)
        if layer.relu:
            a = a.relu()
    loss = F.cross_entropy(a, torch.from_numpy(inputs["labels"]).long())
    # the gradients hang on decisions at ties (see tolerance): they have no one value to be held to
    return dict(logits=a.detach(), loss=loss.detach(), grads=[None] * len(leaves))


def exact(case, seed):
    if case["kind"] == "conv":
        return _exact_conv(case, seed)
    if case["kind"] == "net":
        return _exact_net(case, seed)
    if case["kind"] == "fc":
        x, w, b, dy = (t.double() for t in _fc_tensors(case, seed))
        y = torch.mm(x, w.t().contiguous()) + b
        return dict(y=y.clamp(min=0) if case["relu"] else y, dw=torch.mm(dy.t().contiguous(), x), db=dy.sum(0),
                    dx=torch.mm(dy, w))
    if case["kind"] == "pool":
        x, dy = (t.double() for t in _pool_tensors(case, seed))
        x.requires_grad_()
        if case["mode"] == "max":
            y, _ = F.max_pool2d(x, case["win"], case["stride"], return_indices=True)
        else:
            y = F.avg_pool2d(x, case["win"], case["stride"])
        y.backward(dy)
        # (equal maxima, zeros after the rectifier above all, leave the routed gradient to the tie rule)
        out = dict(y=y.detach(), dx=None if case["mode"] == "max" else x.grad)
        if case["mode"] == "max":
            out["argmax"] = None
        return out
    x, col_in = (t.double() for t in _unroll_tensors(case, seed))
    n, c, h, w, r, s = (case[q] for q in "nchwrs")
    pad = (case["ph"], case["pw"])
    col = F.unfold(x, (r, s), padding=pad)
    cin = col_in.reshape(c * r * s, n, -1).permute(1, 0, 2).contiguous()
    return dict(col=col.permute(1, 0, 2).reshape(c * r * s, -1), dx=F.fold(cin, (h, w), (r, s), padding=pad))
