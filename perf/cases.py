"""Performance cases of the library: what a program that runs a network over video has it do, frame by frame.

A case is one layer (or one stack of layers) with its stored state, in the middle of a video; a pass hands it the next
frame.  The frames of a state are walked forth and back (0, 1, .., K-1, K-2, .., 0, ..), so that every pass sees the
change between two neighbouring frames of the video, however many passes are made.  Values, change patterns and
layer sizes are those of the package's own configurations: post-ReLU activations, square blocks of positions that are
re-drawn between frames, random entries of a feature vector, clustered sign flips, a textured patch moving over a
static background.

Fields of a case
  kind    "stack"  int8 AlexNet-shaped stack of five convolutions through stack_step
          "conv"   one convolution, dtype "i8" or "bf16"        "bin"  one binary convolution
          "fc"     one fully-connected layer, dtype "i8" or "bf16"
  mode    "step"   one frame through Layer.step (difference with the stored input, sparse update)
          "dense"  the plain layer through Layer.dense (a video's first frame, a scene cut, a stateless caller)
  n       independent video streams; h, w, c_in, c_out, k, stride, pad, groups: the layer
  frac    share of the positions (binary: values; FC: entries) that change from one frame to the next
  block   side of the blocks that change
  eps     truncation threshold of a bf16 step; the frames then carry noise below it on every entry
  copy    the step also fills the caller's own output tensor
"""
import math

import numpy as np
import torch

import paper_1802_09723_amd as rrm

FRAMES = 6

# name, h, w, c_in, c_out, k, stride, pad, groups, pooled afterwards
STACK = (
    (227, 227, 3, 96, 11, 4, 0, 1, True),
    (27, 27, 96, 256, 5, 1, 2, 2, True),
    (13, 13, 256, 384, 3, 1, 1, 1, False),
    (13, 13, 384, 384, 3, 1, 1, 1, False),
    (13, 13, 384, 256, 3, 1, 1, 1, False),
)
# share of each layer's input positions that the moving patch changes in a frame
STACK_CHANGE = (0.05, 0.12, 0.30, 0.44, 0.58)


def _conv(name, dtype, mode, n, h, w, c_in, c_out, k, stride, pad, groups, frac, block, eps=0.0, copy=False):
    return dict(name=name, kind="conv", dtype=dtype, mode=mode, n=n, h=h, w=w, c_in=c_in, c_out=c_out, k=k, stride=stride, pad=pad,
                groups=groups, frac=frac, block=block, eps=eps, copy=copy)


def _fc(name, dtype, mode, n, c_in, c_out, frac, copy=False):
    return dict(name=name, kind="fc", dtype=dtype, mode=mode, n=n, c_in=c_in, c_out=c_out, frac=frac, copy=copy)


def listed():
    return [
        # the smallest call: one small int8 layer on one live video; launches and host time are all there is
        _conv("conv_tiny_live_i8", "i8", "step", 1, 32, 32, 16, 16, 3, 1, 1, 1, 0.10, 4),
        # a ResNet-shaped layer on one live video: latency
        _conv("conv_live_bf16", "bf16", "step", 1, 14, 14, 256, 256, 3, 1, 1, 1, 0.05, 8),
        # the early ResNet-shaped layer over many streams of a video archive
        _conv("conv_streams_bf16", "bf16", "step", 64, 56, 56, 64, 64, 3, 1, 1, 1, 0.10, 8),
        # an odd map and channel counts off the powers of two, sensor noise on every entry, truncated by the threshold
        _conv("conv_odd_noise_bf16", "bf16", "step", 9, 35, 29, 80, 112, 3, 1, 1, 1, 0.10, 8, eps=1e-2),
        # the first frame of a few videos: the grouped 5x5 int8 layer, recomputed everywhere
        _conv("conv_first_frame_i8", "i8", "dense", 16, 27, 27, 96, 256, 5, 1, 2, 2, 0.10, 4),
        # a whole stack on one live video: frame rate of a single camera
        dict(name="stack_live_i8", kind="stack", n=1, groups45=1),
        # the same stack over many streams at once: throughput of an archive or a camera farm (the largest case)
        dict(name="stack_streams_i8", kind="stack", n=512, groups45=1),
        # fully-connected layers behind such a stack, one live video: a few entries of the features change
        _fc("fc_live_i8", "i8", "step", 1, 9216, 4096, 0.05),
        # a quarter of the features changes, and the program takes a copy of the result for itself
        _fc("fc_live_copy_bf16", "bf16", "step", 1, 4096, 4096, 0.25, copy=True),
        # many streams share one pass over the weights
        _fc("fc_streams_bf16", "bf16", "step", 64, 9216, 4096, 0.10),
        # XNOR-style layers: one live video, and many streams
        dict(name="bin_live", kind="bin", mode="step", n=1, h=14, w=14, c_in=512, c_out=512, k=3, stride=1, pad=1, groups=1,
             frac=0.10, block=4),
        dict(name="bin_streams", kind="bin", mode="step", n=64, h=28, w=28, c_in=256, c_out=256, k=3, stride=1, pad=1, groups=1,
             frac=0.05, block=4),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _channels(rng, lo, hi):
    """mostly whole 16s, some 8s, some as they come"""
    c = _log(rng, lo, hi)
    step = rng.choice((16, 16, 16, 8, 1))
    return int(min(hi, max(step, round(c / step) * step)))


def draw(rng):
    kind = rng.choices(("conv", "stack", "fc", "bin"), (45, 15, 22, 18))[0]
    if kind == "stack":
        return dict(kind="stack", n=int(round(_log(rng, 1, 512))), groups45=rng.choice((1, 1, 2)))
    mode = "step" if rng.random() < 0.75 else "dense"
    copy = mode == "step" and rng.random() < 0.2
    n = int(round(_log(rng, 1, 64)))
    if kind == "fc":
        dtype = rng.choice(("i8", "bf16"))
        c_in = int(round(_log(rng, 512, 9216)))
        c_out = int(round(_log(rng, 256, 4096)))
        if rng.random() < 0.7:
            c_in, c_out = max(64, c_in // 64 * 64), max(16, c_out // 16 * 16)
        return dict(kind="fc", dtype=dtype, mode=mode, n=int(round(_log(rng, 1, 128))), c_in=c_in, c_out=c_out,
                    frac=round(_log(rng, 0.01, 0.25), 4), copy=copy)
    while True:
        h, w = int(round(_log(rng, 7, 64))), int(round(_log(rng, 7, 64)))
        if rng.random() < 0.5:
            w = h
        k = rng.choice((1, 3, 3, 3, 3, 5))
        stride = rng.choice((1, 1, 1, 2))
        groups = rng.choice((1, 1, 1, 2))
        case = dict(kind=kind, mode=mode, n=n, h=h, w=w, k=k, stride=stride, pad=k // 2, groups=groups)
        if kind == "conv":
            case.update(dtype=rng.choice(("i8", "bf16")), c_in=_channels(rng, 16, 512), c_out=_channels(rng, 16, 512),
                        frac=round(_log(rng, 0.02, 0.5), 4), block=rng.choice((4, 8)), eps=0.0, copy=copy)
            if case["dtype"] == "bf16" and mode == "step" and rng.random() < 0.25:
                case["eps"] = 1e-2
        else:
            case.update(c_in=32 * groups * max(1, int(round(_log(rng, 64, 512) / 32 / groups))), c_out=_channels(rng, 64, 512),
                        frac=round(_log(rng, 0.01, 0.2), 4), block=4)
        if case["c_in"] % groups or case["c_out"] % groups:
            continue
        ho, wo = _out(case)
        macs = case["n"] * ho * wo * case["c_out"] * k * k * case["c_in"] // groups
        if (macs <= 30e9 and case["n"] * h * w * case["c_in"] <= 24e6 and case["n"] * ho * wo * case["c_out"] <= 32e6
                and case["c_out"] * k * k * case["c_in"] // groups <= 5e6):
            return case


def _out(c):
    return (c["h"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1, (c["w"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1


# ---- inputs ----------------------------------------------------------------------------------------------------


class _View:
    """a device buffer as a torch tensor (no copy)"""

    def __init__(self, ptr, shape, typestr):
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": tuple(shape), "typestr": typestr, "version": 2}


def _state_views(layer, x_shape, x_type, y_type):
    """the layer's stored projection and input; the tensors keep the layer, which owns the memory"""
    xp, yp = layer.snapshot_ptrs()
    views = (torch.as_tensor(_View(yp, layer.y_shape, y_type), device="cuda"),
             torch.as_tensor(_View(xp, x_shape, x_type), device="cuda"))
    for v in views:
        v.layer = layer
    return views


def _host(t):
    """a device tensor as the host array that Layer takes (bf16: its 16-bit patterns)"""
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).cpu().numpy().view(np.uint16)
    if t.dtype == torch.int32:
        return t.cpu().numpy().view(np.uint32)
    return t.cpu().numpy()


def _weights(gen, dtype, shape):
    if dtype == "i8":
        return _host(torch.randint(-127, 128, shape, generator=gen, device="cuda", dtype=torch.int8))
    return _host((torch.randn(shape, generator=gen, device="cuda") * 0.05).to(torch.bfloat16))


def _bias(gen, dtype, n):
    if dtype == "i8":
        return torch.randint(-1000, 1001, (n,), generator=gen, device="cuda", dtype=torch.int32).cpu().numpy()
    return (torch.randn((n,), generator=gen, device="cuda") * 0.1).cpu().numpy()


def _act(gen, dtype, shape):
    if dtype == "i8":
        return torch.randint(0, 128, shape, generator=gen, device="cuda", dtype=torch.int8)
    return torch.randn(shape, generator=gen, device="cuda").clamp_(min=0).to(torch.bfloat16)


def _squares(c, frac):
    """(side, count) of the squares whose union covers about `frac` of a map"""
    hw = c["h"] * c["w"]
    side = min(c["block"], c["h"], c["w"])
    if side * side > frac * hw:
        side = max(1, int(math.sqrt(frac * hw)))
    return side, max(1, int(round(math.log(1 - frac) / math.log(1 - side * side / hw))))


def _square_mask(gen, c, frac):
    """[n, h, w]: positions under randomly placed squares"""
    n, h, w = c["n"], c["h"], c["w"]
    side, count = _squares(c, frac)
    y0 = torch.randint(0, h - side + 1, (count, n, 1, 1), generator=gen, device="cuda")
    x0 = torch.randint(0, w - side + 1, (count, n, 1, 1), generator=gen, device="cuda")
    ys = torch.arange(h, device="cuda").view(1, h, 1)
    xs = torch.arange(w, device="cuda").view(1, 1, w)
    mask = torch.zeros((n, h, w), dtype=torch.bool, device="cuda")
    for k in range(count):
        mask |= (ys >= y0[k]) & (ys < y0[k] + side) & (xs >= x0[k]) & (xs < x0[k] + side)
    return mask


def _conv_frames(gen, c):
    shape = (c["n"], c["h"], c["w"], c["c_in"])
    base = _act(gen, c["dtype"], shape)
    frames = []
    for _ in range(FRAMES):
        if frames:
            base = torch.where(_square_mask(gen, c, c["frac"]).unsqueeze(-1), _act(gen, c["dtype"], shape), base)
        frame = base
        if c["eps"]:  # noise well below the threshold in most entries
            frame = (base.float() + 0.15 * c["eps"] * torch.randn(shape, generator=gen, device="cuda")).clamp_(min=0).to(torch.bfloat16)
        frames.append(frame.contiguous())
    return frames


def _fc_frames(gen, c):
    shape = (c["n"], c["c_in"])
    if c["dtype"] == "i8":
        cur = torch.randint(-127, 128, shape, generator=gen, device="cuda", dtype=torch.int8).clamp_(min=0)
    else:
        cur = _act(gen, "bf16", shape)
    frames = [cur]
    k = max(1, int(math.ceil(c["frac"] * c["c_in"])))
    for _ in range(FRAMES - 1):
        pick = torch.rand(shape, generator=gen, device="cuda").argsort(dim=1)[:, :k]
        old = frames[-1].gather(1, pick)
        if c["dtype"] == "i8":
            new = torch.randint(-127, 128, pick.shape, generator=gen, device="cuda", dtype=torch.int8).clamp_(min=0)
            new = torch.where(new == old, (old + 1).clamp_(min=0), new)  # (127 + 1 wraps to a negative value: 0)
        else:
            new = _act(gen, "bf16", pick.shape)
            new = torch.where(new == old, (torch.randn(pick.shape, generator=gen, device="cuda").abs() + 0.01).to(torch.bfloat16), new)
        frames.append(frames[-1].scatter(1, pick, new).contiguous())
    return frames


def _bits(gen, shape):
    return torch.randint(-(1 << 31), 1 << 31, shape, generator=gen, device="cuda", dtype=torch.int64).to(torch.int32)


def _bin_frames(gen, c):
    shape = (c["n"], c["h"], c["w"], c["c_in"] // 32)
    frames = [_bits(gen, shape)]
    for _ in range(FRAMES - 1):  # half of the values under a square flip
        mask = _square_mask(gen, c, min(0.95, 2 * c["frac"])).unsqueeze(-1)
        frames.append(torch.where(mask, frames[-1] ^ _bits(gen, shape), frames[-1]).contiguous())
    return frames


def _stack_frames(gen, rng, n, count):
    """static background, one textured patch of 30..60 pixels per stream moving 1..4 pixels a frame, reflecting"""
    h, w, ch = STACK[0][:3]
    bg = _act(gen, "i8", (n, h, w, ch))
    tex = _act(gen, "i8", (n, 60, 60, ch))
    side = rng.integers(30, 61, n)
    pos = np.stack([rng.uniform(0, h - side), rng.uniform(0, w - side)])
    ang = rng.uniform(0, 2 * math.pi, n)
    step = np.stack([np.sin(ang), np.cos(ang)])
    top = np.stack([h - side, w - side])
    ys = torch.arange(h, device="cuda").view(1, h, 1)
    xs = torch.arange(w, device="cuda").view(1, 1, w)
    which = torch.arange(n, device="cuda").view(n, 1, 1)
    sd = torch.from_numpy(side).cuda().view(n, 1, 1)
    frames = []
    for _ in range(count):
        at = torch.from_numpy(np.rint(np.clip(pos, 0, top)).astype(np.int64)).cuda().view(2, n, 1, 1)
        dy, dx = ys - at[0], xs - at[1]
        inside = (dy >= 0) & (dy < sd) & (dx >= 0) & (dx < sd)
        patch = tex[which, dy.clamp(0, 59), dx.clamp(0, 59)]
        frames.append(torch.where(inside.unsqueeze(-1), patch, bg).contiguous())
        pos = pos + step * rng.integers(1, 5, n)
        for over in (pos < 0, pos > top):
            step = np.where(over, -step, step)
        pos = np.where(pos < 0, -pos, np.where(pos > top, 2 * top - pos, pos))
    return frames


# ---- states and passes -----------------------------------------------------------------------------------------


class _State:
    """a layer or stack, the frames of its video and where in it the program is"""

    def __init__(self, frames):
        self.frames = frames
        self.order = list(range(1, len(frames))) + list(range(len(frames) - 2, -1, -1))
        self.at = 0

    def next_frame(self):
        f = self.frames[self.order[self.at]]
        self.at = (self.at + 1) % len(self.order)
        return f


def _prepare_stack(case, gen, seed):
    n = case["n"]
    s = _State(_stack_frames(gen, np.random.default_rng(seed), n, FRAMES))
    s.layers, s.shifts, s.pools = [], [], []
    x = s.frames[0]
    outs = []
    for i, (h, w, ci, co, k, stride, pad, g, pool) in enumerate(STACK):
        g = case["groups45"] if i >= 3 else g
        layer = rrm.Layer(rrm.Shape(rrm.CONV, n, h, w, ci, co, k, k, stride, pad, g), rrm.I8,
                          _weights(gen, "i8", (co, k, k, ci // g)), _bias(gen, "i8", co))
        # the right shift that brings the layer's largest values to int8, from the first stream's first frame
        y = torch.empty(layer.y_shape, dtype=torch.int32, device="cuda")
        layer.dense(x, y)
        v = y[0].flatten().clamp(min=0)
        top = int(v.kthvalue(max(1, int(math.ceil(0.999 * v.numel()))))[0])
        shift = max(0, top.bit_length() - 7)
        ho, wo = layer.y_shape[1:3]
        po, qo = ((ho - 3) // 2 + 1, (wo - 3) // 2 + 1) if pool else (ho, wo)
        f = torch.empty((n, po, qo, co), dtype=torch.int8, device="cuda")
        rrm.relu_requant_pool_i8(y, f, n, ho, wo, co, shift, pool)
        yv, xv = _state_views(layer, x.shape, "|i1", "<i4")
        outs += [yv, xv]
        s.layers.append(layer)
        s.shifts.append(shift)
        s.pools.append(pool)
        x = f
    s.f_out = x
    s.out = [s.f_out] + outs
    rrm.stack_step(s.layers, s.shifts, s.pools, s.frames[0], s.f_out)
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "stack":
        s = _prepare_stack(case, gen, seed)
        s.stack, s.dense = True, False
        return s
    if case["kind"] == "fc":
        s = _State(_fc_frames(gen, case))
        shape = rrm.Shape(rrm.FC, case["n"], 1, 1, case["c_in"], case["c_out"], 1, 1, 1, 0, 1)
        w_shape, dtype = (case["c_out"], case["c_in"]), case["dtype"]
    else:
        dtype = case.get("dtype", "bin")
        s = _State(_bin_frames(gen, case) if dtype == "bin" else _conv_frames(gen, case))
        k, g = case["k"], case["groups"]
        shape = rrm.Shape(rrm.CONV, case["n"], case["h"], case["w"], case["c_in"], case["c_out"], k, k, case["stride"], case["pad"], g)
        w_shape = (case["c_out"], k, k, case["c_in"] // g)
    if dtype == "bin":
        w = _host(_bits(gen, w_shape[:3] + (w_shape[3] // 32,)))
        s.layer = rrm.Layer(shape, rrm.BIN, w, _bias(gen, "i8", case["c_out"]))
    else:
        s.layer = rrm.Layer(shape, rrm.I8 if dtype == "i8" else rrm.BF16, _weights(gen, dtype, w_shape), _bias(gen, dtype, case["c_out"]))
    if case.get("eps"):
        s.layer.set_threshold(case["eps"])
    s.stack = False
    s.dense = case["mode"] == "dense"
    y_type = torch.float32 if dtype == "bf16" else torch.int32
    s.y = torch.empty(s.layer.y_shape, dtype=y_type, device="cuda") if s.dense or case.get("copy") else None
    if s.dense:
        s.out = s.y
    else:
        yv, xv = _state_views(s.layer, s.frames[0].shape, {"i8": "|i1", "bf16": "<i2", "bin": "<i4"}[dtype],
                              "<f4" if dtype == "bf16" else "<i4")
        s.out = [yv, xv] if s.y is None else [yv, xv, s.y]
        s.layer.step(s.frames[0])  # the video's first frame
    return s


def run(state):
    x = state.next_frame()
    if state.stack:
        rrm.stack_step(state.layers, state.shifts, state.pools, x, state.f_out)
    elif state.dense:
        state.layer.dense(x, state.y)
    else:
        state.layer.step(x, state.y)
    return state.out


def exact(case, seed):
    """The first pass's outputs in 64 bits, from the same draws as prepare's.  Integer layers are compared as they are; of
    a bf16 layer the projection (and the program's own copy of it) is b + W * (the stored input), the stored input after
    a step holds the entries of frame 1 that differ from it by the threshold or more."""
    if case.get("dtype") != "bf16":
        return None
    gen = torch.Generator(device="cuda").manual_seed(seed)
    fc = case["kind"] == "fc"
    frames = _fc_frames(gen, case) if fc else _conv_frames(gen, case)
    k, g = (1, 1) if fc else (case["k"], case["groups"])
    ci, co = case["c_in"] // g, case["c_out"]
    w = _weights(gen, "bf16", (co, ci) if fc else (co, k, k, ci))
    bias = torch.from_numpy(_bias(gen, "bf16", co)).cuda().double()
    w = torch.from_numpy(w.view(np.int16)).cuda().view(torch.bfloat16).double().view(co, k * k, ci)
    x = frames[1]
    if case["mode"] == "step" and case.get("eps"):
        x = torch.zeros_like(frames[0])
        for f in frames[:2]:
            # (the difference is decided in fp32, the precision in which the library states the threshold)
            x = torch.where((f.float() - x.float()).abs() >= np.float32(case["eps"]).item(), f, x)
    if fc:
        y = x.double() @ w[:, 0].t() + bias
    else:
        n, st, pad = case["n"], case["stride"], case["pad"]
        ho, wo = _out(case)
        xp = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
        og = co // g
        y = bias.expand(n * ho * wo, co).clone()
        for t in range(k * k):
            ky, kx = divmod(t, k)
            part = xp[:, ky:ky + st * (ho - 1) + 1:st, kx:kx + st * (wo - 1) + 1:st]
            for i in range(g):
                cols = part[..., i * ci:(i + 1) * ci].reshape(-1, ci).contiguous()
                y[:, i * og:(i + 1) * og] += cols @ w[i * og:(i + 1) * og, t].t().contiguous()
        y = y.view(n, ho, wo, co)
    if case["mode"] == "dense":
        return y
    return [y, None, y] if case.get("copy") else [y, None]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------


def _cover(c, frac, reach):
    """share of the map under the changed squares, each grown by `reach` positions"""
    side, count = _squares(c, frac)
    p = min(side + reach, c["h"]) * min(side + reach, c["w"]) / (c["h"] * c["w"])
    return 1 - (1 - min(p, 1.0)) ** count


def work(case):
    """a step reads the frame and the stored input, writes the stored input where it changed, reads the weights and
    reads and writes the projection where a changed input reaches it; products: those of the changed inputs"""
    if case["kind"] == "stack":
        n, by, fl = case["n"], 0.0, 0.0
        for i, (h, w, ci, co, k, stride, pad, g, pool) in enumerate(STACK):
            g = case["groups45"] if i >= 3 else g
            ho, wo = (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1
            ch = STACK_CHANGE[i]
            reach = min(1.0, ch * 1.5)  # changed outputs
            x, y = n * h * w * ci, n * ho * wo * co
            by += (2 if i == 0 else ch) * x + ch * x + co * k * k * ci // g + 8 * reach * y
            by += 4 * reach * y  # the map to the next layer's input
            fl += 2.0 * ch * y * k * k * ci // g
        return {"bytes": by, "flops": fl}
    esize = {"i8": 1, "bf16": 2}.get(case.get("dtype"), 0.125)
    if case["kind"] == "fc":
        x, y, wgt, per = case["n"] * case["c_in"], case["n"] * case["c_out"], case["c_in"] * case["c_out"], case["c_in"]
        changed, reached = case["frac"], 1.0
        used = 1 - (1 - changed) ** case["n"]  # columns of the weights
    else:
        ho, wo = _out(case)
        per = case["k"] * case["k"] * case["c_in"] // case["groups"]
        x, y, wgt = case["n"] * case["h"] * case["w"] * case["c_in"], case["n"] * ho * wo * case["c_out"], case["c_out"] * per
        used = 1.0
        changed = case["frac"]
        reached = _cover(case, min(0.95, 2 * changed) if case["kind"] == "bin" else changed, case["k"] - 1)
    if case["mode"] == "dense":
        return {"bytes": esize * (x + wgt) + 4.0 * y, "flops": 2.0 * y * per}
    by = esize * (2 * x + changed * x + used * wgt) + 8.0 * reached * y
    if case.get("copy"):
        by += 4.0 * (2 - reached) * y  # all of it is written once more, and what did not change is read
    return {"bytes": by, "flops": 2.0 * changed * y * per}


def tolerance(case):
    # int8 and binary layers are integer arithmetic; bf16 layers add exact products in fp32, in any order, and carry a
    # difference as two bf16 terms
    if case.get("dtype") == "bf16":
        return {"rel": 1e-5}
    return "exact"
