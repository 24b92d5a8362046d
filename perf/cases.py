"""Workloads whose time matters: what a detector's training and inference programs ask of this library.

Every case runs through the public calls of ``paper_1903_05831_amd`` on one stream.  The layers of a
case are isolated operators with tensors of their own, as in ``bench.py``: a forward pass over all
layers, then, in training, the data gradient and the weight gradient of each layer from the last to
the first, then the removal of the loss scale with its overflow check, and the optimizer step where
the case has one.  Layer shapes are those of a ResNet-50-C4 / ResNet-50-FPN Faster R-CNN
(``workloads.py``) on images and numbers of RoIs of any size.
"""
from __future__ import annotations

import math
from typing import NamedTuple

import torch

import paper_1903_05831_amd as sd


class Layer(NamedTuple):
    part: str       # outputs of one part of the network lie in one buffer
    N: int
    H: int
    W: int
    C: int
    K: int
    R: int
    stride: int = 1
    pad: int = 0
    dil: int = 1
    shortcut: bool = False      # last convolution of a residual block: the shortcut is added to it
    relu: bool = True

    @property
    def out_hw(self):
        def ext(n):
            return (n + 2 * self.pad - self.dil * (self.R - 1) - 1) // self.stride + 1
        return ext(self.H), ext(self.W)

    @property
    def x_shape(self):
        return self.N, self.H, self.W, self.C

    @property
    def w_shape(self):
        return self.K, self.R, self.R, self.C

    @property
    def y_shape(self):
        return (self.N, *self.out_hw, self.K)

    @property
    def desc(self):
        return sd.make_desc(self.N, self.H, self.W, self.C, self.K, self.R, self.R, (self.stride,) * 2,
                            (self.pad,) * 2, (self.dil,) * 2)


def _half(n):
    return (n - 1) // 2 + 1


def _stage(part, N, H, W, cin, mid, blocks, stride, project=True):
    """Bottleneck blocks 1x1, 3x3, 1x1 (expansion 4); the first one has the stride and, where the
    shape changes, the 1x1 projection."""
    out, cout = [], 4 * mid
    for b in range(blocks):
        s = stride if b == 0 else 1
        out.append(Layer(part, N, H, W, cin, mid, 1))
        out.append(Layer(part, N, H, W, mid, mid, 3, s, 1))
        h, w = (_half(H), _half(W)) if s == 2 else (H, W)
        out.append(Layer(part, N, h, w, mid, cout, 1, shortcut=True))
        if b == 0 and project:
            out.append(Layer(part, N, H, W, cin, cout, 1, s, relu=False))
        H, W, cin = h, w, cout
    return out


def _stem(N, h, w):
    return [Layer("stem", N, h, w, 3, 64, 7, 2, 3)]


def _backbone(N, h, w):
    h4, w4 = _half(_half(h)), _half(_half(w))
    h8, w8 = _half(h4), _half(w4)
    return (_stem(N, h, w) + _stage("res2", N, h4, w4, 64, 64, 3, 1) + _stage("res3", N, h4, w4, 256, 128, 4, 2)
            + _stage("res4", N, h8, w8, 512, 256, 6, 2))


def _roi_head(rois):
    return _stage("res5", rois, 14, 14, 1024, 512, 3, 2)


def _fpn(N, h, w):
    out, maps = [], []
    h, w = _half(_half(h)), _half(_half(w))
    for c in (256, 512, 1024, 2048):
        maps.append((h, w))
        out.append(Layer("lateral", N, h, w, c, 256, 1, relu=False))
        h, w = _half(h), _half(w)
    out += [Layer("output", N, h, w, 256, 256, 3, 1, 1, relu=False) for h, w in maps]
    maps.append((_half(maps[-1][0]), _half(maps[-1][1])))
    for h, w in maps:
        out += [Layer("rpn", N, h, w, 256, 256, 3, 1, 1),
                Layer("objectness", N, h, w, 256, 3, 1, relu=False), Layer("boxes", N, h, w, 256, 12, 1, relu=False)]
    return out


def _c4_rpn(N, h, w):
    return [Layer("rpn", N, h, w, 1024, 512, 3, 1, 1),
            Layer("objectness", N, h, w, 512, 15, 1, relu=False), Layer("boxes", N, h, w, 512, 60, 1, relu=False)]


def _layers(case):
    net, N = case["net"], case["N"]
    h, w = case.get("H", 1), case.get("W", 1)
    if net == "conv":
        return [Layer("conv", N, h, w, case["C"], case["K"], case["R"], case["stride"], case["pad"], case["dil"])]
    if net == "res2":       # a later block of the stage: no projection
        return _stage("res2", N, h, w, 256, 64, case["blocks"], 1, project=False)
    if net == "res3":
        return _stage("res3", N, h, w, 256, 128, case["blocks"], 2)
    if net == "res4":
        return _stage("res4", N, h, w, 512, 256, case["blocks"], 2)
    if net == "stem":
        return _stem(N, h, w)
    if net == "backbone":
        return _backbone(N, h, w)
    if net == "roi_head":
        return _roi_head(N)
    if net == "fpn":
        return _fpn(N, h, w)
    if net == "c4_rpn":
        return _c4_rpn(N, h, w)
    if net == "box_head":   # two fully connected layers on 7x7x256 RoI features
        return [Layer("fc6", N, 1, 1, 7 * 7 * 256, 1024, 1), Layer("fc7", N, 1, 1, 1024, 1024, 1)]
    if net == "detector":
        return _backbone(N, h, w) + _roi_head(case["rois"])
    raise ValueError(net)


def listed():
    return [
        # the smallest convolution, one image: launches and latency
        dict(name="conv3x3_small_train", net="conv", mode="train", fused=False, dtype="fp16",
             N=1, H=56, W=56, C=64, K=64, R=3, stride=1, pad=1, dil=1),
        # a high-resolution bottleneck: few channels, memory-bound 1x1 layers
        dict(name="res2_block_train", net="res2", mode="train", fused=False, dtype="fp16", N=2, H=200, W=336, blocks=1),
        # a strided first block with frozen-BN tails on a map of odd size (one image of 692x1084)
        dict(name="res3_block_train_odd", net="res3", mode="train", fused=True, dtype="fp16", N=1, H=173, W=271, blocks=1),
        # the trunk that holds most layers of the backbone
        dict(name="res4_trunk_train", net="res4", mode="train", fused=False, dtype="fp16", N=2, H=100, W=168, blocks=6),
        # second stage of the C4 detector on a training step's RoIs: the large matrix products
        dict(name="roi_head_train", net="roi_head", mode="train", fused=True, dtype="fp16", N=512),
        # the same head in inference, on the proposals that are left of one image
        dict(name="roi_head_infer", net="roi_head", mode="infer", fused=True, dtype="fp16", N=100),
        # inference of the backbone on one image whose sides are no multiple of anything
        dict(name="backbone_infer_odd", net="backbone", mode="infer", fused=True, dtype="fp16", N=1, H=750, W=1333),
        # pyramid and RPN heads over five levels: many small layers, 3 and 12 filters
        dict(name="fpn_rpn_train", net="fpn", mode="train", fused=False, dtype="fp16", N=2, H=800, W=1344),
        # box head: fully connected layers, a long contraction on few rows
        dict(name="box_head_train", net="box_head", mode="train", fused=True, dtype="fp16", N=512),
        # loss scale, overflow check and SGD over the weights of the detector
        dict(name="optimizer_tail", net="optimizer", mode="update", n=23454912, overflow=False),
        # full precision, for comparison runs: one strided res4 block
        dict(name="res4_block_fp32_train", net="res4", mode="train", fused=False, dtype="fp32", N=1, H=100, W=168, blocks=1),
        # everything: one training step of the C4 detector with its optimizer step
        dict(name="detector_step", net="detector", mode="step", fused=False, dtype="fp16", N=2, H=800, W=1344, rois=512),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv", "conv", "res2", "res3", "res4", "roi_head", "roi_head", "backbone", "fpn", "box_head",
                       "optimizer", "fp32", "detector", "stem", "c4_rpn"])
    case = dict(net=kind, mode=rng.choice(["train", "train", "infer"]), fused=rng.random() < 0.5, dtype="fp16")
    N = rng.choice([1, 1, 2, 2, 3, 4])
    h, w = rng.randint(400, 800), rng.randint(500, 1344)
    if kind == "conv":
        dil = rng.choice([1, 1, 1, 2])
        R = rng.choice([1, 3, 3])
        case.update(mode="train", N=N, H=_spread(rng, 14, 200), W=_spread(rng, 14, 336), C=8 * _spread(rng, 4, 64),
                    K=8 * _spread(rng, 4, 64), R=R, stride=rng.choice([1, 1, 2]), pad=dil if R == 3 else 0, dil=dil)
        if work(case)["flops"] > 1e12:
            case["N"] = 1
    elif kind in ("res2", "res3"):
        case.update(N=N, H=_half(_half(h)), W=_half(_half(w)), blocks=rng.randint(1, 3))
    elif kind == "res4":
        case.update(N=N, H=_half(_half(_half(h))), W=_half(_half(_half(w))), blocks=rng.randint(1, 6))
    elif kind == "roi_head":
        case.update(N=_spread(rng, 20, 512))
    elif kind == "box_head":
        case.update(N=_spread(rng, 50, 1024))
    elif kind == "backbone":
        case.update(N=rng.choice([1, 2]), H=h, W=w)
    elif kind in ("fpn", "stem"):
        case.update(N=min(N, 2), H=h, W=w)
    elif kind == "c4_rpn":
        case.update(N=N, H=_half(_half(_half(_half(h)))), W=_half(_half(_half(_half(w)))))
    elif kind == "detector":
        case.update(mode="step", N=1, H=h, W=w, rois=rng.randint(64, 256))
    elif kind == "fp32":
        case.update(net=rng.choice(["res2", "res3", "res4"]), mode="train", fused=False, dtype="fp32", N=1,
                    H=rng.randint(40, 120), W=rng.randint(60, 168), blocks=1)
    else:
        case = dict(net="optimizer", mode="update", n=_spread(rng, 100_000, 30_000_000), overflow=rng.random() < 0.2)
    return case


LOSS_SCALE = 1024.0
LR, MOMENTUM, WEIGHT_DECAY, GROWTH, BACKOFF, INTERVAL = 0.02, 0.9, 1e-4, 2.0, 0.5, 2000


def _normal(gen, shape, dtype, sigma=1.0):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, sigma, generator=gen)


def _optimizer_state(gen, n):
    master = _normal(gen, n, torch.float32, 0.05)
    scale = torch.zeros(2, dtype=torch.int32, device="cuda")
    scale[:1].view(torch.float32).fill_(LOSS_SCALE)
    return dict(master=master, momentum=_normal(gen, n, torch.float32, 1e-3), w_half=torch.empty_like(master, dtype=torch.float16),
                flag=torch.zeros(1, dtype=torch.int32, device="cuda"), scale=scale)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    state = dict(case=case)
    if case["mode"] == "update":
        # gradients of about 1e-3 times the loss scale (a later pass meets the unscaled ones)
        state.update(_optimizer_state(gen, case["n"]), grad=_normal(gen, case["n"], torch.float32))
        if case["overflow"]:
            state["grad"][torch.randint(case["n"], (1 + case["n"] // 10_000,), device="cuda", generator=gen)] = math.inf
        return state

    layers = _layers(case)
    dtype = torch.float16 if case["dtype"] == "fp16" else torch.float32
    train = case["mode"] != "infer"
    parts = list(dict.fromkeys(l.part for l in layers))

    def buffers(shape_of, dtype):
        """One buffer for each part of the network, and the layers' tensors in it (256-byte aligned)."""
        whole, views = {}, [None] * len(layers)
        for part in parts:
            own = [i for i, l in enumerate(layers) if l.part == part]
            sizes = [math.prod(shape_of(layers[i])) for i in own]
            offs = [0]
            for n in sizes:
                offs.append(offs[-1] + -(-n // 128) * 128)
            whole[part] = torch.zeros(offs[-1], dtype=dtype, device="cuda")
            for i, n, o in zip(own, sizes, offs):
                views[i] = whole[part][o:o + n].view(shape_of(layers[i]))
        return whole, views

    y_all, y = buffers(lambda l: l.y_shape, dtype)
    ops, sizes = [], [math.prod(l.w_shape) for l in layers]
    if train:
        dx_all, dx = buffers(lambda l: l.x_shape, dtype)
        offs = [0]
        for n in sizes:
            offs.append(offs[-1] + -(-n // 128) * 128)
        dw_all = torch.zeros(offs[-1], dtype=torch.float32, device="cuda")
        state.update(dx_all=dx_all, dw_all=dw_all, flag=torch.zeros(1, dtype=torch.int32, device="cuda"))
    state.update(ops=ops, y_all=y_all)
    workspace_bytes = sd.conv2d_workspace_bytes if case["dtype"] == "fp16" else sd.conv2d_workspace_bytes_f32
    need = 256
    for i, l in enumerate(layers):
        d = l.desc
        op = dict(desc=d, y=y[i], x=_normal(gen, l.x_shape, dtype),
                  w=_normal(gen, l.w_shape, dtype, math.sqrt(2.0 / (l.R * l.R * l.C))))
        if case["fused"]:
            if l.C > 3:
                op["x"].relu_()     # the activation of the layer before
            op["relu"] = l.relu
            op["fwd_scale"] = _normal(gen, l.K, torch.float32, 0.25).add_(1.0)
            op["fwd_bias"] = _normal(gen, l.K, torch.float32)
            op["shortcut"] = _normal(gen, l.y_shape, dtype) if l.shortcut else None
            op["bwd_scale"] = _normal(gen, l.C, torch.float32, 0.25).add_(1.0)
        if train:
            op.update(dy=_normal(gen, l.y_shape, dtype), dx=dx[i], dw=dw_all[offs[i]:offs[i] + sizes[i]].view(l.w_shape))
        need = max([need] + [workspace_bytes(d, p) for p in ((sd.FWD, sd.DGRAD, sd.WGRAD) if train else (sd.FWD,))])
        ops.append(op)
    state["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    if case["mode"] == "step":
        state.update(_optimizer_state(gen, dw_all.numel()))
    return state


def run(state):
    case, st = state["case"], torch.cuda.current_stream().cuda_stream
    if case["mode"] == "update":
        _update(state, state["grad"], st)
        return [state[k] for k in ("grad", "master", "momentum", "w_half", "flag", "scale")]
    ws, fused = state["workspace"], case["fused"]
    if case["dtype"] == "fp16":
        fwd, dgrad, wgrad = sd.conv2d_fwd, sd.conv2d_dgrad, sd.conv2d_wgrad
    else:
        fwd, dgrad, wgrad = sd.conv2d_fwd_f32, sd.conv2d_dgrad_f32, sd.conv2d_wgrad_f32
    for o in state["ops"]:
        if fused:
            sd.conv2d_fwd_fused(o["desc"], o["x"], o["w"], o["y"], ws, st, scale=o["fwd_scale"], bias=o["fwd_bias"],
                                residual=o["shortcut"], relu=o["relu"])
        else:
            fwd(o["desc"], o["x"], o["w"], o["y"], ws, st)
    out = list(state["y_all"].values())
    if case["mode"] == "infer":
        return out
    for o in reversed(state["ops"]):
        if fused:
            sd.conv2d_dgrad_fused(o["desc"], o["dy"], o["w"], o["dx"], ws, st, scale=o["bwd_scale"], relu_mask=o["x"])
        else:
            dgrad(o["desc"], o["dy"], o["w"], o["dx"], ws, st)
        wgrad(o["desc"], o["x"], o["dy"], o["dw"], ws, st)
    dw = state["dw_all"]
    out += [*state["dx_all"].values(), dw, state["flag"]]
    if case["mode"] == "step":
        _update(state, dw, st)
        return out + [state[k] for k in ("master", "momentum", "w_half", "scale")]
    sd.grad_unscale_check(dw, dw.numel(), 1.0 / LOSS_SCALE, state["flag"], st)
    return out


def _update(s, grad, st):
    sd.grad_unscale_check_dynamic(grad, grad.numel(), s["scale"], s["flag"], st)
    sd.sgd_momentum_update(s["master"], s["momentum"], grad, s["w_half"], grad.numel(), LR, MOMENTUM, WEIGHT_DECAY,
                           s["flag"], s["scale"], GROWTH, BACKOFF, INTERVAL, st)


def work(case):
    """Each call on its own: its inputs read once, its outputs written once."""
    unscale, update = 8, 22     # bytes an element
    if case["mode"] == "update":
        return dict(bytes=(unscale + update) * case["n"], flops=8 * case["n"])
    size = 2 if case["dtype"] == "fp16" else 4
    nbytes = flops = 0
    for l in _layers(case):
        x, w, y = math.prod(l.x_shape), math.prod(l.w_shape), math.prod(l.y_shape)
        passes = 1 if case["mode"] == "infer" else 3
        flops += passes * 2 * y * l.R * l.R * l.C
        nbytes += size * (x + w + y)
        if case["fused"] and l.shortcut:
            nbytes += size * y
        if passes == 3:
            nbytes += size * (x + w + y) + size * (x + y) + 4 * w + unscale * w
            if case["fused"]:
                nbytes += size * x
        if case["mode"] == "step":
            nbytes += update * w
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["mode"] == "update":
        return "exact"      # every operation is defined, one rounding each
    if case["dtype"] == "fp32":
        # measured against sums in 64 bits: rel 4.0e-7, max 3.1e-6; four times that and a little
        # for contractions longer than the measured ones
        return dict(rel=2e-6, max=2e-5)
    # one rounding of a binary32 sum to binary16: rel 2.1e-4 and max 4.9e-4 against the same sums in
    # 64 bits, and one step of 2^-10 where two orders of a sum round apart
    return dict(rel=8e-4, max=4e-3)
