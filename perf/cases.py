"""The calls a user of this library makes, over the sizes it is used at.

A case is a dict of plain values; `prepare` makes what a program holds before the call (frames in device memory, the
pipeline or layer handle, planted detector heads), `run` is one pass through the public entry points and returns what it
computes.  Three kinds of call:

  cascade  frames -> letterbox -> detector -> decode / top-k / NMS -> ROI table -> crop-resize -> children -> results, as
           a serving program drives it: submit, run, collect (binding.Pipeline).  The networks are those of zoo.py, the
           scenes those of synth.py (uniform-noise background, filled rectangles), made on the GPU.  Random weights cannot
           detect a prescribed scene, so, as in the benchmark, the tensors that decode reads are planted
           (Pipeline.set_head), except for the tiny fp32 network, whose own heads are used.
  conv     one convolution layer on caller-owned tensors (binding.op_conv).
  stages   the stage calls in a row on caller-owned tensors, for a program that runs a detector of its own:
           letterbox, decode, top-k, NMS, ROI compaction, crop-resize.
"""
from __future__ import annotations

import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2502_01277_amd import binding, synth, zoo

# Colours of the objects.  A camera sees the same kinds of object again and again; with a handful of appearances the
# classes of the crops are also decided by more than the rounding of a 16-bit logit.
PALETTE = [(24, 136, 136), (24, 24, 80), (24, 136, 184), (232, 80, 80), (184, 80, 184), (184, 232, 232), (80, 184, 136), (80, 24, 136)]

# Networks: builder of the pipeline description, per-frame object counts, sides of the objects at the source's scale
# (fractions of the frame height), most ROIs a frame may have, low-score candidates beside the objects.
NETS = {
    "tiny":         dict(counts="fixed", mean=6.0, sides=(0.05, 0.30), rois=100, clutter=0, classes=8),
    "traffic":      dict(counts="poisson", mean=8.0, sides=(0.022, 0.33), rois=64, clutter=0, classes=80),
    "sweep":        dict(counts="negbin", mean=6.0, sides=(0.022, 0.185), rois=200, clutter=0, classes=80),
    "surveillance": dict(counts="poisson", mean=8.0, sides=(0.022, 0.33), rois=64, clutter=0, classes=80),
    "detonly":      dict(counts="poisson", mean=8.0, sides=(0.022, 0.33), rois=64, clutter=0, classes=80),
    "hires":        dict(counts="pareto", mean=14.0, sides=(0.022, 0.33), rois=300, clutter=1100, classes=80),
}


def listed():
    return [
        # two small frames, fp32, a network of five layers and a classifier of five: nothing but latency
        dict(name="tiny_f32_2", kind="cascade", net="tiny", dtype="f32", frames=2, capacity=2, instances=1, src_h=320, src_w=320),
        # one camera, one frame at a time, answered as soon as possible
        dict(name="sweep_bf16_1", kind="cascade", net="sweep", dtype="bf16", frames=1, capacity=1, instances=1, src_h=1080, src_w=1920),
        # the traffic cascade with both children, one batch at a time
        dict(name="traffic_f16_8", kind="cascade", net="traffic", dtype="f16", frames=8, capacity=8, instances=1, src_h=1080, src_w=1920),
        # the same with four instances of the pipeline on streams of their own, a batch each, as the benchmark runs it
        dict(name="traffic_f16_8x4", kind="cascade", net="traffic", dtype="f16", frames=8, capacity=8, instances=4, src_h=1080, src_w=1920),
        # people surveillance: bottleneck attribute classifier on upright crops
        dict(name="surveillance_bf16_16", kind="cascade", net="surveillance", dtype="bf16", frames=16, capacity=16, instances=1, src_h=1080, src_w=1920),
        # detector only, a batch that is not full, frames of a camera whose size is no multiple of anything
        dict(name="detonly_f16_5of16", kind="cascade", net="detonly", dtype="f16", frames=5, capacity=16, instances=1, src_h=769, src_w=1366),
        # the batch size with the best throughput of the sweep
        dict(name="sweep_bf16_64", kind="cascade", net="sweep", dtype="bf16", frames=64, capacity=64, instances=1, src_h=1080, src_w=1920),
        # the largest configuration: 32 frames of 3840 x 2160, thousands of ROIs
        dict(name="hires_bf16_32", kind="cascade", net="hires", dtype="bf16", frames=32, capacity=32, instances=1, src_h=2160, src_w=3840),
        # one layer: a classifier stage in 8-bit floating point at a served batch
        dict(name="conv_f8_3x3", kind="conv", dtype="f8", n=1021, h=14, w=14, cin=256, cout=256, k=3, stride=1, act=zoo.ACT_RELU, res=zoo.RES_BEFORE_ACT),
        # one layer: a wide map of the high-resolution detector through a 1x1 convolution, bound by memory
        dict(name="conv_bf16_1x1", kind="conv", dtype="bf16", n=32, h=160, w=160, cin=96, cout=96, k=1, stride=1, act=zoo.ACT_SILU, res=zoo.RES_NONE),
        # one layer: a down-sampling 3x3 on a few images of odd size
        dict(name="conv_f16_3x3s2", kind="conv", dtype="f16", n=9, h=57, w=83, cin=96, cout=192, k=3, stride=2, act=zoo.ACT_SILU, res=zoo.RES_NONE),
        # the stage calls around a detector of the user's own
        dict(name="stages_bf16_8", kind="stages", net="traffic", dtype="bf16", frames=8, src_h=1080, src_w=1920),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_source(rng, lo, hi):
    """Height and width of a camera frame: any size between the two heights, aspect ratios from 4:3 to 16:9."""
    h = _log_int(rng, lo, hi)
    return dict(src_h=h, src_w=int(h * rng.uniform(1.3, 1.8)))


def draw(rng):
    pick = rng.random()
    half = rng.choice(["f16", "bf16"])
    if pick < 0.10:
        n = rng.randint(1, 4)
        return dict(kind="cascade", net="tiny", dtype="f32", frames=n, capacity=n, instances=1, **_draw_source(rng, 240, 480))
    if pick < 0.60:
        net = rng.choice(["sweep", "traffic", "surveillance", "detonly"])
        n = _log_int(rng, 1, {"sweep": 64, "traffic": 32, "surveillance": 24, "detonly": 64}[net])
        inst = rng.choice([1, 1, 1, 2, 3, 4]) if n <= 12 else 1
        cap = n if rng.random() < 0.7 else min(64, n + rng.randint(1, 8))
        return dict(kind="cascade", net=net, dtype=half, frames=n, capacity=cap, instances=inst, **_draw_source(rng, 480, 1440))
    if pick < 0.66:
        n = _log_int(rng, 1, 24)
        return dict(kind="cascade", net="hires", dtype=half, frames=n, capacity=n, instances=1, **_draw_source(rng, 1080, 2160))
    if pick < 0.92:
        while True:
            k = rng.choice([1, 1, 3, 3])
            stride = rng.choice([1, 1, 2])
            dtype = rng.choice(["f16", "bf16", "f8", "f32"])
            step = {"f8": 16, "f16": 8, "bf16": 8, "f32": 4}[dtype]
            h = _log_int(rng, 7, 160)
            c = dict(kind="conv", dtype=dtype, n=_log_int(rng, 1, 2048), h=h, w=max(7, int(h * rng.uniform(0.6, 1.5))),
                     cin=step * max(1, _log_int(rng, 16, 768) // step), cout=8 * max(1, _log_int(rng, 16, 768) // 8), k=k, stride=stride,
                     act=rng.choice([zoo.ACT_RELU, zoo.ACT_SILU]), res=rng.choice([zoo.RES_NONE, zoo.RES_NONE, zoo.RES_BEFORE_ACT, zoo.RES_AFTER_ACT]))
            w = work(c)
            if 1e8 < w["flops"] < (8e10 if dtype == "f32" else 1.5e12) and w["bytes"] < 1e9:
                return c
    return dict(kind="stages", net="traffic", dtype=half, frames=_log_int(rng, 1, 32), **_draw_source(rng, 480, 1440))


# ---- inputs -----------------------------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _models(net, dtype):
    """The network's description with its weights.  Weights belong to the program, not to a pass: one seed for all."""
    if net == "tiny":
        p = zoo.tiny_cascade(dtype)
        # the benchmark's tiny detector finds about a hundred objects in a frame; this one about as many as its scene has
        det = zoo.plain_detector("tiny_det", dtype, 320, (16, 32, 64, 128), 8, zoo.SEED0 + 1, batch_size=2, score_thr=0.25, iou_thr=0.45,
                                 topk=100, max_det=100, obj_bias=-1.0)
        return dataclasses.replace(p, models=[det] + p.models[1:])
    return {"traffic": zoo.traffic_cascade, "surveillance": zoo.surveillance_cascade, "detonly": zoo.detector_only, "hires": zoo.hires_cascade,
            "sweep": lambda dtype: zoo.sweep_cascade(8, dtype)}[net](dtype=dtype)


def _spec(case):
    base, cap, rois = _models(case["net"], case["dtype"]), case.get("capacity", case["frames"]), NETS[case["net"]]["rois"]
    models = [dataclasses.replace(m, batch_size=cap if i == 0 else cap * rois) for i, m in enumerate(base.models)]
    return dataclasses.replace(base, models=models, src_h=case["src_h"], src_w=case["src_w"], max_frames=cap, max_rois_per_frame=rois)


def _scene(rng, net, n, h, w):
    """Per object: frame, corners in source pixels, class."""
    p = NETS[net]
    if p["counts"] == "fixed":
        counts = np.full(n, int(p["mean"]))
    else:
        counts = {"poisson": lambda: synth.counts_poisson(rng, n, p["mean"], p["rois"]), "negbin": lambda: synth.counts_negbin(rng, n),
                  "pareto": lambda: synth.counts_pareto(rng, n)}[p["counts"]]()
    f = np.repeat(np.arange(n), counts)
    lo, hi = np.log(np.array(p["sides"]) * h)
    sw, sh = (np.minimum(np.floor(np.exp(rng.uniform(lo, hi, f.size))), s - 1) for s in (w, h))
    x1, y1 = np.floor(rng.random(f.size) * (w - sw)), np.floor(rng.random(f.size) * (h - sh))
    return f, np.stack([x1, y1, x1 + sw, y1 + sh], 1), rng.integers(0, p["classes"], f.size)


def _frames(rng, gen, n, h, w, f, rect):
    """uint8 [n][h][w][3]: uniform noise, the objects in their colour with a little of the noise left as texture."""
    x = torch.randint(0, 256, (n, h, w, 3), dtype=torch.uint8, device="cuda", generator=gen)
    colours = (torch.tensor(PALETTE, dtype=torch.int16) - 16).clamp_(0, 223).to(torch.uint8).cuda()
    which = rng.integers(0, len(PALETTE), f.size)
    for j in range(f.size):
        x1, y1, x2, y2 = (int(v) for v in rect[j])
        x[f[j], y1:y2, x1:x2].bitwise_right_shift_(3).add_(colours[which[j]])
    return list(x)


def _logit(p):
    return np.log(p / (1.0 - p))


def _planted_heads(rng, gen, det, net, n, src_h, src_w, f, rect, cls):
    """Head tensors whose decode yields the scene's objects, up to four near-duplicates of each for NMS to remove, and
    (high-resolution network) more low-score candidates than top-k keeps, crowded around forty spots a frame."""
    A, C, size = det.n_anchors, det.n_classes, det.in_w
    no = 5 + C
    dt = binding.torch_dtype(det.dtype)
    heads = []
    for g in det.grids:
        t = torch.randn((n, g * g, A, no), dtype=dt, device="cuda", generator=gen).mul_(1.5)
        t[..., 5:].clamp_(max=2.0)
        t[..., 4] = -8.0
        heads.append(t)
    nw, nh, left, top = binding.letterbox_geometry(src_h, src_w, det.in_h, det.in_w)
    cx, cy = (rect[:, 0] + rect[:, 2]) / 2 * (nw / src_w) + left, (rect[:, 1] + rect[:, 3]) / 2 * (nh / src_h) + top
    bw, bh = np.maximum((rect[:, 2] - rect[:, 0]) * nw / src_w, 2.0), np.maximum((rect[:, 3] - rect[:, 1]) * nh / src_h, 2.0)
    anchors, strides = det.anchors.astype(np.float64).reshape(-1, 2), np.array(det.strides)
    inter = np.minimum(bw[:, None], anchors[None, :, 0]) * np.minimum(bh[:, None], anchors[None, :, 1])
    best = (inter / (bw[:, None] * bh[:, None] + anchors.prod(1)[None] - inter)).argmax(1) if f.size else np.zeros(0, int)
    lvl, an = best // A, best % A
    gx, gy = np.floor(cx / strides[lvl]), np.floor(cy / strides[lvl])
    obj = rng.uniform(1.0, 4.0, f.size)
    rows = [(f, lvl, an, gx, gy, cx, cy, bw, bh, obj, cls)]
    dups = rng.integers(0, 5, f.size)
    for d in range(4):
        m = dups > d
        k = int(m.sum())
        kind = rng.random(k)                                # another anchor of the cell, the cell beside it, the cell above or below
        a2 = np.where(kind < 0.5, (an[m] + 1 + rng.integers(0, A - 1, k)) % A, an[m])
        dx = np.where(cx[m] / strides[lvl[m]] - gx[m] < 0.5, -1, 1) * ((kind >= 0.5) & (kind < 0.75))
        dy = np.where(cy[m] / strides[lvl[m]] - gy[m] < 0.5, -1, 1) * (kind >= 0.75)
        rows.append((f[m], lvl[m], a2, gx[m] + dx, gy[m] + dy, cx[m], cy[m], bw[m] * rng.uniform(0.9, 1.1, k), bh[m] * rng.uniform(0.9, 1.1, k),
                     obj[m] - rng.uniform(0.2, 1.0, k), cls[m]))
    k = int(NETS[net]["clutter"] * 1.4)                     # some fall on a taken slot or outside what an anchor can express
    if k:
        spot = rng.integers(0, 40, (n, k))
        at = lambda lo, hi: np.take_along_axis(rng.uniform(lo, hi, (n, 40)) * size, spot, 1).ravel()   # noqa: E731
        sx, sy, sw, sh = at(0.1, 0.9), at(0.25, 0.75), at(0.05, 0.18), at(0.05, 0.18)
        scls = np.take_along_axis(rng.integers(0, C, (n, 40)), spot, 1).ravel()
        m = n * k
        ux, uy = sx + rng.uniform(-0.25, 0.25, m) * sw, sy + rng.uniform(-0.25, 0.25, m) * sh
        ul = rng.integers(0, len(det.grids), m)
        target = rng.uniform(0.262, 0.298, m) * (1.0 + math.exp(-4.0))        # score = sigmoid(obj) * sigmoid(4)
        rows.append((np.repeat(np.arange(n), k), ul, rng.integers(0, A, m), np.floor(ux / strides[ul]), np.floor(uy / strides[ul]), ux, uy,
                     sw * rng.uniform(0.85, 1.15, m), sh * rng.uniform(0.85, 1.15, m), _logit(target), scls))
    f, lvl, an, gx, gy, cx, cy, bw, bh, obj, cls = (np.concatenate(v) for v in zip(*rows))
    s, g, a2 = strides[lvl], np.array(det.grids)[lvl], anchors[lvl * A + an]
    p = np.stack([((cx / s - gx) + 0.5) / 2, ((cy / s - gy) + 0.5) / 2, np.sqrt(bw / a2[:, 0]) / 2, np.sqrt(bh / a2[:, 1]) / 2], 1)
    ok = ((p > 0.02) & (p < 0.98)).all(1) & (gx >= 0) & (gy >= 0) & (gx < g) & (gy < g)
    slot = ((f * len(det.grids) + lvl) * (g * g) + gy * g + gx).astype(np.int64) * A + an
    first = np.zeros(slot.size, bool)
    idx = np.flatnonzero(ok)
    first[idx[np.unique(slot[idx], return_index=True)[1]]] = True
    v = np.concatenate([_logit(np.clip(p, 0.01, 0.99)), obj[:, None], np.full((p.shape[0], C), -6.0)], 1)
    v[np.arange(v.shape[0]), 5 + cls] = 4.0
    for l, t in enumerate(heads):
        m = np.flatnonzero(first & (lvl == l))
        if m.size:
            at = [torch.from_numpy(np.ascontiguousarray(q[m]).astype(np.int64)).cuda() for q in (f, gy * g + gx, an)]
            t[at[0], at[1], at[2]] = torch.from_numpy(v[m].astype(np.float32)).cuda().to(dt)
    return [t.view(n, g, g, A * no) for t, g in zip(heads, det.grids)]


class _Streams:
    """One stream per instance over all compute units, given back with the state."""

    def __init__(self, n):
        cus = binding.device_cu_count()
        self.handles = [binding.stream_create_range(0, cus) for _ in range(n)]

    def __del__(self):
        for h in self.handles:
            binding.stream_destroy(h)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return {"cascade": _prepare_cascade, "conv": _prepare_conv, "stages": _prepare_stages}[case["kind"]](case, rng, gen)


def _prepare_cascade(case, rng, gen):
    spec, n = _spec(case), case["frames"]
    parts, keep = [], _Streams(case["instances"]) if case["instances"] > 1 else None
    for i in range(case["instances"]):
        f, rect, cls = _scene(rng, case["net"], n, case["src_h"], case["src_w"])
        P = binding.Pipeline(spec)
        heads = None
        if case["net"] != "tiny":
            heads = _planted_heads(rng, gen, spec.models[0], case["net"], n, case["src_h"], case["src_w"], f, rect, cls)
            for l, t in enumerate(heads):
                P.set_head(0, l, t)
        parts.append((P, _frames(rng, gen, n, case["src_h"], case["src_w"], f, rect), keep.handles[i] if keep else None, heads))
    torch.cuda.synchronize()                      # the instances' streams are not torch's
    return dict(kind="cascade", parts=parts, streams=keep)


def _prepare_conv(case, rng, gen):
    dtype, n, h, w, cin, cout, k = (case[v] for v in ("dtype", "n", "h", "w", "cin", "cout", "k"))
    K = k * k * cin
    bias = rng.uniform(-0.1, 0.1, cout).astype(np.float32)
    scale = None
    if dtype == "f8":
        raw = synth.e4m3_codes(rng, (cout, k, k, cin))
        scale = np.full(cout, 0.5 / math.sqrt(K), np.float32)
    else:
        raw = synth.to_storage(rng.standard_normal((cout, k, k, cin), dtype=np.float32) * np.float32(math.sqrt(2.0 / K)), dtype)
    layer = binding.ConvOp(raw, bias, dtype, case["stride"], k // 2, case["act"], scale=scale)
    ho, wo = layer.out_hw(h, w)

    def tensor(*shape):
        if dtype != "f8":
            return torch.randn(shape, dtype=binding.torch_dtype(dtype), device="cuda", generator=gen)
        t = torch.randint(0, 0x48, shape, dtype=torch.uint8, device="cuda", generator=gen)            # magnitudes up to 3.75
        return t.bitwise_or_(torch.randint(0, 2, shape, dtype=torch.uint8, device="cuda", generator=gen).bitwise_left_shift_(7))

    x = tensor(n, h, w, cin)
    y = torch.empty((n, ho, wo, cout), dtype=x.dtype, device="cuda")
    return dict(kind="conv", layer=layer, x=x, y=y, res=tensor(n, ho, wo, cout) if case["res"] else None, res_mode=case["res"])


def _prepare_stages(case, rng, gen):
    spec, n = _spec(case), case["frames"]
    det, crop = spec.models[0], spec.models[1]
    f, rect, cls = _scene(rng, case["net"], n, case["src_h"], case["src_w"])
    heads = _planted_heads(rng, gen, det, case["net"], n, case["src_h"], case["src_w"], f, rect, cls)
    return dict(kind="stages", det=det, crop=(crop.in_h, crop.in_w), heads=heads, frames=_frames(rng, gen, n, case["src_h"], case["src_w"], f, rect),
                src=(case["src_h"], case["src_w"]), cap=16 * n)                  # crops its classifier takes


# ---- one pass -----------------------------------------------------------------------------------------------------------
def _table(rows, cap):
    """Result records in a table of fixed length (the program's own), as numbers: floats and whole values of a record."""
    t = np.zeros(cap, rows.dtype)
    t[:len(rows)] = rows
    return t.view(np.float32).reshape(cap, 8), t.view(np.int32).reshape(cap, 8)


def run(state):
    if state["kind"] == "conv":
        s = state
        binding.op_conv(s["layer"], s["x"], s["y"], s["res"], s["res_mode"], res_scale=1.0, y_inv_scale=1.0)
        return s["y"]
    if state["kind"] == "cascade":
        for P, frames, stream, _ in state["parts"]:
            P.submit(frames)
            P.run(stream)
        out = []
        for P, _, _, _ in state["parts"]:
            fr, bx, _ = P.collect()
            f, i = _table(bx, len(fr) * P.spec.models[0].max_det)            # corners, score | class, labels of the children
            out.append([fr["frame_id"], fr["n_boxes"], fr["flags"], f[:, :5], i[:, 5:]])
        return out
    det, frames = state["det"], state["frames"]
    x = binding.op_letterbox(frames, det.in_h, det.in_w, det.dtype)
    cand, count = binding.op_decode(det, state["heads"])
    top, n_top = binding.op_topk(cand, count, min(det.topk, det.n_cand()))
    keep, n_keep = binding.op_nms(top, n_top, det.iou_thr, det.max_det)
    rois, roi_of, boxes, flags = binding.op_compact(top, keep, n_keep, state["src"], (det.in_h, det.in_w), (1 << 128) - 1, state["cap"])
    crops = binding.op_crop_resize(frames, rois, *state["crop"], det.dtype, cap=state["cap"])
    rf, ri = _table(rois, state["cap"])
    bf, bi = _table(boxes.reshape(-1), boxes.size)
    return [x, count, n_top, keep, n_keep, roi_of, flags, ri[:, :3], rf[:, 4:], bf[:, :5], bi[:, 5:], crops]


# ---- what a pass cannot do without, and how near two correct ones are ------------------------------------------------------
def work(case):
    es = {"f32": 4, "f16": 2, "bf16": 2, "f8": 1}[case["dtype"]]
    if case["kind"] == "conv":
        s, p = case["stride"], case["k"] // 2
        ho, wo = ((case[d] + 2 * p - case["k"]) // s + 1 for d in ("h", "w"))
        y = case["n"] * ho * wo * case["cout"]
        taps = case["k"] ** 2 * case["cin"]
        read = case["n"] * case["cin"] * (ho * wo if case["k"] < s else case["h"] * case["w"])     # a strided 1x1 layer skips pixels
        return dict(bytes=es * (read + y * (2 if case["res"] else 1) + case["cout"] * taps), flops=2.0 * y * taps)
    base, n = _models(case["net"], case["dtype"]), case["frames"] * case.get("instances", 1)
    det = base.models[0]
    # source pixels: each output pixel of the letterbox needs at most four, and there are no more than the frame has
    r = min(det.in_h / case["src_h"], det.in_w / case["src_w"])
    shown = case["src_h"] * case["src_w"] * r * r
    pixels = 3.0 * min(case["src_h"] * case["src_w"], 4 * shown) * n
    heads = 0.0 if case["net"] == "tiny" else es * n * det.n_cand() * (5 + det.n_classes)
    p = NETS[case["net"]]
    rois = n * min(p["rois"], p["mean"] + p["clutter"] / 10)
    if case["kind"] == "stages":
        crop = base.models[1]
        return dict(bytes=pixels + heads + es * (n * det.in_h * det.in_w * 3 + rois * crop.in_h * crop.in_w * 3), flops=0.0)
    weights = sum(L.weight.size for m in base.models for L in m.layers if L.weight is not None)
    return dict(bytes=pixels + heads + es * weights * case["instances"],
                flops=n * det.flops_per_item() + rois * sum(m.flops_per_item() for m in base.models[1:]))


def tolerance(case):
    if case["kind"] == "conv":
        # one rounding of the result to its type, which fp32 sums in another order move now and then; 8-bit results are codes
        return {"f32": dict(rel=1e-5), "f16": dict(rel=1e-3), "bf16": dict(rel=5e-3), "f8": dict(rel=1e-5, differ=0.01)}[case["dtype"]]
    if case["kind"] == "stages":
        return dict(rel=5e-3 if case["dtype"] == "bf16" else 1e-3, differ=0.0)
    # boxes are decoded in fp32 from given heads (the tiny network's own are fp32 too); labels are the largest of up to
    # a thousand 16-bit-network logits, whose first two are now and then closer than the roundings on the way
    return dict(rel=1e-5, differ=0.01)
