"""Measured cases: the work a user has the library do, through its public calls.

A case is a dict of plain values.  ``kind`` names the path, the other values
its sizes and options:

    crops   crops of u8 BGR (or NV12) frames, resized, normalised, planar fp32:
            ``frames`` frames of ``fw`` x ``fh``, ``batch`` crops with sides
            ``lo``..``hi``, outputs ``ow`` x ``oh`` (0 x 0: each 224 x 224 or
            64 x 128, as the serving requests mix them)
    depth   one frame, cvt and ``n_ops`` alternating scalar mul / add, packed
    ops     a chain of ``n_ops`` random ops over a batch of frames
    cast    a batch of 60 x 120 one-channel images: cast, mul, sub, div
    stats   per-channel min, max, sum and mean of a batch of frames
    mlp     the cost model's network: forward, loss, backward

Chains and their constants follow from the case (``ops_seed``); pixels, crop
rectangles, weights and features follow from the seed of the inputs.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2508_07071_amd as fk

NP = {"u8": np.uint8, "f16": np.float16, "f32": np.float32, "f64": np.float64}
MEAN, STD = (0.485, 0.456, 0.406), (0.229, 0.224, 0.225)
OUT_SIZES = ((64, 128), (128, 128), (224, 224), (256, 256), (512, 512))
DEV = "cuda"


def listed() -> list:
    return [
        # the smallest call: one detection resized for a classifier; launch and latency
        {"name": "one_crop", "kind": "crops", "read": "crop_resize", "frames": 1, "fw": 1920, "fh": 1080,
         "batch": 1, "lo": 512, "hi": 512, "ow": 224, "oh": 224},
        # a frame's detections in one launch (64 wide x 128 high, uneven sides)
        {"name": "crops_256", "kind": "crops", "read": "crop_resize", "frames": 1, "fw": 3840, "fh": 2160,
         "batch": 256, "lo": 60, "hi": 600, "ow": 64, "oh": 128},
        # a serving loop's coalesced launch: many requests, two output sizes
        {"name": "crops_served", "kind": "crops", "read": "crop_resize", "frames": 24, "fw": 3840, "fh": 2160,
         "batch": 778, "lo": 60, "hi": 600, "ow": 0, "oh": 0},
        # the same detections on a video decoder's frame
        {"name": "crops_nv12", "kind": "crops", "read": "nv12_resize", "frames": 1, "fw": 3840, "fh": 2160,
         "batch": 256, "lo": 60, "hi": 600, "ow": 64, "oh": 128},
        # a large frame through a short chain (HBM) and through a long one (arithmetic)
        {"name": "depth_16", "kind": "depth", "dtype": "u8", "channels": 3, "fw": 3840, "fh": 2160, "n_ops": 16,
         "out": "f32", "ops_seed": 1},
        {"name": "depth_256", "kind": "depth", "dtype": "u8", "channels": 3, "fw": 3840, "fh": 2160, "n_ops": 256,
         "out": "f32", "ops_seed": 2},
        # chains known only at run time, as the cost model's chains are drawn:
        # whole frames, and crops resized to a half-precision network input
        {"name": "ops_plain", "kind": "ops", "read": "plain", "dtype": "f16", "channels": 3, "fw": 1501, "fh": 1103,
         "batch": 9, "ow": 0, "oh": 0, "n_ops": 37, "out": "f32", "layout": "planar", "ops_seed": 3},
        {"name": "ops_resize", "kind": "ops", "read": "crop_resize", "dtype": "u8", "channels": 3, "fw": 1920,
         "fh": 1080, "batch": 48, "ow": 256, "oh": 256, "n_ops": 29, "out": "f16", "layout": "planar", "ops_seed": 4},
        # many small images in one launch
        {"name": "cast_600", "kind": "cast", "dtype": "u8", "out": "f32", "batch": 600, "ops_seed": 5},
        # image statistics of a batch of frames
        {"name": "stats_16", "kind": "stats", "dtype": "u8", "channels": 3, "fw": 3840, "fh": 2160, "batch": 16},
        # a chain computed in double
        {"name": "double_64", "kind": "depth", "dtype": "f32", "channels": 3, "fw": 3840, "fh": 2160, "n_ops": 64,
         "out": "f64", "ops_seed": 6},
        # one mini-batch of the cost model's training, forward and backward
        {"name": "mlp_512", "kind": "mlp", "rows": 512, "hidden": 128},
    ]


def _logint(r: random.Random, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(r.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random) -> dict:
    """One more case of the listed ones' ranges."""
    kind = rng.choice(("crops", "crops", "depth", "ops", "ops", "cast", "stats", "double", "mlp"))
    if kind == "crops":
        frames = _logint(rng, 1, 24)
        fw, fh = 2 * rng.randint(320, 1920), 2 * rng.randint(240, 1080)
        ow, oh = rng.choice(((0, 0), (224, 224), (64, 128), (rng.randint(33, 300), rng.randint(33, 300))))
        return {"kind": "crops", "read": rng.choice(("crop_resize", "crop_resize", "crop_nearest", "nv12_resize")),
                "frames": frames, "fw": fw, "fh": fh, "batch": _logint(rng, 1, 900), "lo": 60,
                "hi": min(600, fw, fh), "ow": ow, "oh": oh}
    if kind in ("depth", "double"):
        c = rng.choice((1, 3, 4))
        w, h = _logint(rng, 60, 3840), _logint(rng, 60, 2160)
        dt, out = (rng.choice(("u8", "f16", "f32")), "f32") if kind == "depth" else \
                  (rng.choice(("u8", "f16", "f32", "f64")), "f64")
        n = _logint(rng, 1, 256 if kind == "depth" else 64)
        return {"kind": "depth", "dtype": dt, "channels": c, "fw": w, "fh": h, "n_ops": n, "out": out,
                "ops_seed": rng.randrange(1 << 30)}
    if kind == "ops":
        c, dt = rng.choice((1, 3, 4)), rng.choice(("u8", "f16", "f32"))
        case = {"kind": "ops", "read": rng.choice(("plain", "crop_resize")), "dtype": dt, "channels": c,
                "fw": _logint(rng, 64, 2048), "fh": _logint(rng, 64, 2048), "batch": _logint(rng, 1, 256),
                "ow": 0, "oh": 0, "n_ops": rng.randint(1, 64), "out": rng.choice(("f32", "f16")),
                "layout": rng.choice(("packed", "planar")), "ops_seed": rng.randrange(1 << 30)}
        if case["read"] == "crop_resize":
            case["ow"], case["oh"] = rng.choice(OUT_SIZES + ((rng.randint(33, 300), rng.randint(33, 300)),))
        # about the largest listed chain's elements, and frames that are made quickly
        px = max(case["fw"] * case["fh"], case["ow"] * case["oh"])
        case["batch"] = max(1, min(case["batch"], 9 * 1501 * 1103 // px))
        return case
    if kind == "cast":
        dt, out = rng.choice((("u8", "f32"), ("u8", "f16"), ("f16", "f32"), ("f16", "f16"), ("f32", "f32"),
                              ("f32", "f16"), ("f32", "f64"), ("f64", "f64")))
        return {"kind": "cast", "dtype": dt, "out": out, "batch": _logint(rng, 1, 1191),
                "ops_seed": rng.randrange(1 << 30)}
    if kind == "stats":
        dt = rng.choice(("u8", "u8", "f16", "f32"))
        w, h = _logint(rng, 64, 3840), _logint(rng, 64, 2160)
        es = NP[dt]().itemsize
        return {"kind": "stats", "dtype": dt, "channels": rng.choice((1, 3, 4)), "fw": w, "fh": h,
                "batch": max(1, min(_logint(rng, 1, 64), 16 * 3840 * 2160 // (w * h * es)))}
    return {"kind": "mlp", "rows": _logint(rng, 32, 2048), "hidden": rng.choice((128, 128, 64, 96))}


# ------------------------------------------------------------------ inputs --

def _f32(v) -> float:
    return float(np.float32(v))


def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(seed)


def _pixels(g, shape, dtype: str):
    """Uniform random bytes; u8-range values for the other types."""
    if dtype == "u8":
        return torch.randint(0, 256, shape, dtype=torch.uint8, device=DEV, generator=g)
    wide = torch.float64 if dtype == "f64" else torch.float32
    return (torch.rand(shape, dtype=wide, device=DEV, generator=g) * 255.0).to(fk.TORCH_DTYPE[dtype])


def _op(kind, k=()):
    return {"kind": kind, "k": [_f32(v) for v in k]}


def _chain(case: dict) -> dict:
    r = random.Random(case.get("ops_seed", 0))
    kind = case["kind"]
    read = {"kind": case.get("read", "plain"), "dtype": case.get("dtype", "u8"), "channels": case.get("channels", 3),
            "out_w": 0, "out_h": 0}
    if kind == "crops":
        ops = [_op("swap"), _op("cvt"), _op("mul", (1.0 / 255.0,)), _op("sub", MEAN), _op("div", STD)]
        write = {"dtype": "f32", "layout": "planar"}
    elif kind == "depth":
        ops = [_op("cvt")] + [_op("mul", (r.uniform(0.5, 1.5),)) if i % 2 == 0 else _op("add", (r.uniform(-1, 1),))
                              for i in range(case["n_ops"])]
        write = {"dtype": case["out"], "layout": "packed"}
    elif kind == "ops":
        ops = []
        for _ in range(case["n_ops"]):
            k = r.choice(("swap", "cvt", "mul", "add", "sub", "div"))
            n = 0 if k in ("swap", "cvt") else 1 if r.random() < 0.5 else read["channels"]
            lo, hi = (0.5, 1.5) if k in ("mul", "div") else (-1.0, 1.0)
            ops.append(_op(k, [r.uniform(lo, hi) for _ in range(n)]))
        write = {"dtype": case["out"], "layout": case["layout"]}
    elif kind == "cast":
        read["channels"] = 1
        ops = [_op("cvt"), _op("mul", (r.uniform(0.5, 1.5),)), _op("sub", (r.uniform(-1, 1),)),
               _op("div", (r.uniform(0.5, 1.5),))]
        write = {"dtype": case["out"], "layout": "packed"}
    else:
        ops = [_op("cvt")]
        write = {"dtype": "f64", "layout": "stats"}
    return {"read": read, "ops": ops, "write": write}


def _frames(case: dict, seed: int) -> list:
    g = _gen(seed)
    if case["kind"] == "cast":  # columns of up to 512 images of 60 x 120
        b = case["batch"]
        return [_pixels(g, (min(b, 512) * 120, (b + 511) // 512 * 60, 1), case["dtype"])]
    w, h, c, dt = case["fw"], case["fh"], case.get("channels", 3), case.get("dtype", "u8")
    if case.get("read") == "nv12_resize":
        return [_pixels(g, (h * 3 // 2, w), "u8") for _ in range(case["frames"])]
    n = case["frames"] if case["kind"] == "crops" else case.get("batch", 1)
    return [_pixels(g, (h, w, c), dt) for _ in range(n)]


def _items(case: dict, seed: int) -> list:
    r = random.Random(seed)
    sizes = random.Random(case.get("batch", 1))  # the mix of output sizes belongs to the case
    kind = case["kind"]
    if kind == "cast":
        return [{"frame": 0, "x": b // 512 * 60, "y": b % 512 * 120, "w": 60, "h": 120, "out_w": 60, "out_h": 120}
                for b in range(case["batch"])]
    w, h = case["fw"], case["fh"]
    if kind == "crops" or case.get("read") == "crop_resize":
        out = []
        for b in range(case["batch"]):
            lo, hi_w, hi_h = case.get("lo", 16), min(w, case.get("hi", w)), min(h, case.get("hi", h))
            cw, ch = r.randint(min(lo, hi_w), hi_w), r.randint(min(lo, hi_h), hi_h)
            size = (case["ow"], case["oh"]) if case["ow"] else sizes.choice(((224, 224), (64, 128)))
            f = b * case["frames"] // case["batch"] if kind == "crops" else b
            out.append({"frame": f, "x": r.randint(0, w - cw), "y": r.randint(0, h - ch), "w": cw, "h": ch,
                        "out_w": size[0], "out_h": size[1]})
        return out
    return [{"frame": b, "x": 0, "y": 0, "w": w, "h": h, "out_w": w, "out_h": h} for b in range(case.get("batch", 1))]


def _groups(items: list) -> dict:
    """Items by output size, in first-seen order."""
    by: dict = {}
    for i, it in enumerate(items):
        by.setdefault((it["out_w"], it["out_h"]), []).append(i)
    return by


def _mlp_inputs(case: dict, seed: int) -> dict:
    g = _gen(seed)
    n, dims = case["rows"], (fk.FK_MODEL_FEATURES, case["hidden"], case["hidden"], case["hidden"], fk.FK_MODEL_OUTPUTS)
    layers = []
    for a, b in zip(dims[:-1], dims[1:]):  # He-uniform weights, small biases
        s = math.sqrt(6.0 / a)
        layers.append(((torch.rand((b, a), device=DEV, generator=g) * 2 - 1) * s,
                       (torch.rand((b,), device=DEV, generator=g) * 2 - 1) * 0.1))
    x = torch.randn((n, dims[0]), device=DEV, generator=g)                 # standardised features
    t = torch.rand((n, dims[-1]), device=DEV, generator=g).mul_(0.8)       # log-time ratios
    return {"layers": layers, "x": x, "t": t}


class _State:
    """Inputs, outputs and the plan or model handle a program keeps."""

    plan = model = None

    def __del__(self):
        if self.plan:
            fk.fk_plan_destroy(self.plan)
        if self.model:
            fk.fk_model_destroy(self.model)


def prepare(case: dict, seed: int):
    s = _State()
    if case["kind"] == "mlp":
        inp = _mlp_inputs(case, seed)
        n = case["rows"]
        s.x, s.t = inp["x"], inp["t"]
        s.model = fk.fk_model_create(case["hidden"], 0)
        flat = torch.cat([v.reshape(-1) for wb in inp["layers"] for v in wb])
        fk.fk_model_set_params(s.model, flat.cpu().numpy())
        s.ws = torch.empty(fk.fk_mlp_workspace_floats(s.model, n), device=DEV)
        s.y, s.dy = (torch.empty((n, fk.FK_MODEL_OUTPUTS), device=DEV) for _ in range(2))
        s.loss = torch.empty(1, device=DEV)
        s.grad = torch.empty(fk.fk_model_param_count(s.model), device=DEV)
        return s
    chain, items = _chain(case), _items(case, seed)
    s.frames = _frames(case, seed)
    outs, s.out = [None] * len(items), []
    dt = fk.TORCH_DTYPE[chain["write"]["dtype"]]
    for idx in _groups(items).values():  # one tensor per output size
        t = torch.empty((len(idx),) + tuple(fk.out_shape(chain, items[idx[0]])), dtype=dt, device=DEV)
        s.out.append(t)
        for j, i in enumerate(idx):
            outs[i] = t[j]
    s.n = len(items)
    s.desc = fk.chain_desc(chain)
    s.plan = fk.fk_plan_create(s.desc, s.n)
    s.items = fk.make_items(chain, s.frames, items, outs)
    return s


def run(state):
    s = state
    if s.model:
        fk.fk_mlp_forward(s.model, s.x, s.ws, s.y)
        fk.fk_mlp_mse(s.y, s.t, s.dy, s.loss)
        fk.fk_mlp_backward(s.model, s.x, s.ws, s.dy, s.grad)
        return [s.y, s.loss, s.dy, s.grad]
    fk.fk_run(s.plan, s.items, s.n, fk.stream_handle())
    return s.out


# ----------------------------------------------------- necessary work --

def work(case: dict) -> dict:
    if case["kind"] == "mlp":
        n, h = case["rows"], case["hidden"]
        f, o = fk.FK_MODEL_FEATURES, fk.FK_MODEL_OUTPUTS
        params = (f + 1) * h + 2 * (h + 1) * h + (h + 1) * o
        macs = n * (f * h + 2 * h * h + h * o)
        return {"bytes": 4 * (2 * params + n * (f + 3 * o)), "flops": 2 * (3 * macs - n * f * h)}
    chain, items = _chain(case), _items(case, 0)
    c = chain["read"]["channels"]
    es_in, es_out = NP[chain["read"]["dtype"]]().itemsize, NP[chain["write"]["dtype"]]().itemsize
    rk, stats = chain["read"]["kind"], chain["write"]["layout"] == "stats"
    rd = wr = px = 0
    for it in items:
        n = it["out_w"] * it["out_h"]
        taps = 1 if rk == "crop_nearest" else 2
        src = n if rk == "plain" else min(it["w"], taps * it["out_w"]) * min(it["h"], taps * it["out_h"])
        rd += src * 3 // 2 if rk == "nv12_resize" else src * c * es_in
        wr += 32 * c if stats else n * c * es_out
        px += n
    per = sum(op["kind"] in ("mul", "add", "sub", "div") for op in chain["ops"])
    per += 4 if stats else 0 if rk in ("plain", "crop_nearest") else 6
    return {"bytes": rd + wr, "flops": px * c * per}


# ------------------------------------------------------------- exact values --

def _coord(n_out: int, n_in: int):
    """Taps and weight of every output index; the source coordinate is fp32 by definition."""
    scale = float(np.float32(n_in) / np.float32(n_out))
    o = torch.arange(n_out, dtype=torch.float64, device=DEV)
    s = ((o + 0.5) * scale - 0.5).float().clamp_min(0.0).double()
    i0 = s.floor().clamp_max(n_in - 1)
    return i0.long(), (i0 + 1).clamp_max(n_in - 1).long(), s - i0


def _read(case: dict, frame, it: dict):
    x, y, w, h, ow, oh = (it[k] for k in ("x", "y", "w", "h", "out_w", "out_h"))
    rk = case.get("read", "plain")
    if rk == "plain":
        return frame[y:y + h, x:x + w].double()
    if rk == "crop_nearest":
        ix = (2 * torch.arange(ow, device=DEV) + 1) * w // (2 * ow)
        iy = (2 * torch.arange(oh, device=DEV) + 1) * h // (2 * oh)
        return frame[y:y + h, x:x + w][iy][:, ix].double()
    if rk == "nv12_resize":
        fh = case["fh"]
        ys, xs = torch.arange(y, y + h, device=DEV), torch.arange(x, x + w, device=DEV)
        luma = frame[ys][:, xs].double() - 16.0
        uv = frame[fh + ys // 2]
        u, v = uv[:, xs // 2 * 2].double() - 128.0, uv[:, xs // 2 * 2 + 1].double() - 128.0
        k = luma * _f32(1.164)
        roi = torch.stack((k + _f32(2.018) * u, k - _f32(0.813) * v - _f32(0.391) * u, k + _f32(1.596) * v), -1)
    else:
        roi = frame[y:y + h, x:x + w].double()
    x0, x1, ax = _coord(ow, w)
    y0, y1, ay = _coord(oh, h)
    ax, ay = ax[None, :, None], ay[:, None, None]
    top, bot = roi[y0], roi[y1]
    top = top[:, x0] + ax * (top[:, x1] - top[:, x0])
    bot = bot[:, x0] + ax * (bot[:, x1] - bot[:, x0])
    return top + ay * (bot - top)


def _apply(ops: list, v):
    for op in ops:
        kind = op["kind"]
        if kind == "swap":
            if v.shape[-1] >= 3:
                v = v[..., [2, 1, 0] + list(range(3, v.shape[-1]))]
            continue
        if kind == "cvt":
            continue
        k = torch.tensor(op["k"], dtype=torch.float64, device=DEV)
        v = v * k if kind == "mul" else v + k if kind == "add" else v - k if kind == "sub" else v / k
    return v


def exact(case: dict, seed: int):
    if case["kind"] == "mlp":
        inp = _mlp_inputs(case, seed)
        ws = [(w.double(), b.double()) for w, b in inp["layers"]]
        acts = [inp["x"].double()]
        for i, (w, b) in enumerate(ws):
            z = acts[-1] @ w.t() + b
            acts.append(z if i == len(ws) - 1 else z.clamp_min(0.0))
        d = acts[-1] - inp["t"].double()
        loss = (d * d).mean().reshape(1)
        dy = g = d * (2.0 / d.numel())
        grads = []
        for i in reversed(range(len(ws))):
            grads[:0] = [(g.t() @ acts[i]).reshape(-1), g.sum(0)]
            if i:
                g = (g @ ws[i][0]) * (acts[i] > 0)
        return [acts[-1], loss, dy, torch.cat(grads)]
    chain, items = _chain(case), _items(case, seed)
    frames = _frames(case, seed)
    out = []
    for idx in _groups(items).values():
        res = []
        for i in idx:
            v = _apply(chain["ops"], _read(case, frames[items[i]["frame"]], items[i]))
            if chain["write"]["layout"] == "stats":
                f = v.reshape(-1, v.shape[-1])
                total = f.sum(0)
                v = torch.stack((f.amin(0), f.amax(0), total, total / f.shape[0]), -1)
            elif chain["write"]["layout"] == "planar":
                v = v.permute(2, 0, 1).contiguous()
            res.append(v)
        out.append(torch.stack(res))
    return out
