"""Convolutions that do not depend on one another in one launch (conv_small_group_kernel): a shortcut beside its block's first layer, and three 1x1 layers of different inputs and
channel counts.  Every tensor bit for bit what the layers give in launches of their own, with buffers that are kept and with buffers that are reused."""
import numpy as np
import pytest
import torch

import bench
from oracle import nn
from paper_2502_01277_amd import synth, zoo
from helpers import TOL, rel_err, small_root

SMALL = 13


def _launches(kids, g):
    """Of a group's members (tensor numbers): layers of its launch, and ids of the members that had a launch of their own."""
    ids = [kids[t - 1] for t in g]
    one = [k for k in ids if k // 10**7 == 213]
    return (one[0] // 10**6 % 10 // 2 if one else 0), sorted(k // 10**8 for k in ids if k and k // 10**7 != 213), ids.count(0)


def _shortcut(dtype, n, h, w):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(61))
    B.ch = [16]
    B.m.in_c = 16
    x = B.conv(0, 64, 1, act=zoo.ACT_RELU)
    last = []
    for c in (128, 256):
        a = B.conv(x, c, 1, 2, act=zoo.ACT_NONE)
        b = B.conv(x, c, 3, 2, act=zoo.ACT_RELU)
        x = B.conv(b, c, 3, 1, act=zoo.ACT_RELU, res=a, res_mode=zoo.RES_BEFORE_ACT)
        last += [(a, b)]
    B.m.outputs = [B.fc(B.gap(x), 10)]
    B.m.batch_size = n
    return B.m, last


def _heads(dtype, n, h, w):
    B = zoo._Builder("t", dtype, h, w, "classifier", np.random.default_rng(62))
    B.ch = [16]
    B.m.in_c = 16
    t = [B.conv(0, 64, 1, act=zoo.ACT_RELU)]
    for c in (192, 128):
        t.append(B.conv(t[-1], c, 3, act=zoo.ACT_SILU))
    out = tuple(B.conv(s, c, 1, act=zoo.ACT_NONE) for s, c in zip(t, (40, 264, 72)))
    B.m.outputs = [B.fc(B.gap(B.cat(list(out))), 10)]
    B.m.batch_size = n
    return B.m, [out]


PAIR, THREE = ([SMALL] * 2, (2, [])), ([SMALL] * 3, (3, []))
APART = ([SMALL, 20], (0, [SMALL, 20]))                  # the 3x3 layer goes to conv3x3_held_kernel, and the other, collected by itself, is launched as it is


# want: per group the kernels of its layers on their own, and (layers of its launch, kernels of the members that have launches of their own)
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("make,n,h,w,want", [(_shortcut, 1, 9, 11, [PAIR, PAIR]), (_shortcut, 11, 28, 28, [PAIR, APART]), (_shortcut, 40, 41, 39, [PAIR, PAIR]), (_heads, 1, 5, 3, [THREE]),
                                             (_heads, 3, 20, 21, [THREE]), (_heads, 9, 40, 40, [THREE])])
def test_bit_for_bit_what_the_layers_give_alone(octo, dtype, make, n, h, w, want):
    m, groups = make(dtype, n, h, w)
    x = zoo.round_to_dtype(np.random.default_rng(63).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    members = [t for g in groups for t in g]
    got, kids, work = {}, {}, {}
    for keep in (1, 2, 0):
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        for _ in range(2):                               # buffers hold the results of an earlier run
            P.run_model_on(1, octo.to_device(x, dtype))
        got[keep] = {t: P.get_tensor(1, t, n) for t in (members if keep else []) + [m.outputs[0]]}
        kids[keep] = [int(q) for q in P.layer_info(1)[1]]
        work[keep] = [float(v.sum()) for v in P.layer_info(1)[2:]]
        P.close()
    ref = nn.run_model(m, x[:1], keep_all=True)
    for t in members:
        assert rel_err(got[2][t][:1], ref[t]) <= TOL[dtype], t
        assert np.array_equal(got[2][t], got[1][t]), t
    assert np.array_equal(got[0][m.outputs[0]], got[1][m.outputs[0]])
    for g, (alone, fused) in zip(groups, want):
        assert _launches(kids[1], g) == (0, alone, 0), kids[1]
        # the launch is reported by one member, the others of it report none
        count, others, none = _launches(kids[2], g)
        assert (count, others) == fused and none == max(0, count - 1) and count + len(others) == len(g), kids[2]
    assert kids[0] == kids[2]
    assert work[1] == pytest.approx(work[2], rel=1e-12) and work[0] == work[2]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_with_the_count_on_the_device(octo, dtype):
    """A residual classifier downstream, where the pair of shortcut and first layer has its item count on the device: none, a few, more than one round of workgroups and a few again.  Bit for bit
    what the layers give alone, nothing written behind the count, and with timing the launch's time is its first layer's."""
    det = zoo.traffic_cascade(dtype).models[0]
    det.batch_size = 4
    B = zoo._Builder("child", dtype, 64, 64, "classifier", np.random.default_rng(64))
    x = B.conv(0, 64, 3, 2, act=zoo.ACT_RELU)
    members = []
    for c in (128, 256):
        a = B.conv(x, c, 1, 2, act=zoo.ACT_NONE)
        b = B.conv(x, c, 3, 2, act=zoo.ACT_RELU)
        x = B.conv(b, c, 3, 1, act=zoo.ACT_RELU, res=a, res_mode=zoo.RES_BEFORE_ACT)
        members.append((a, b))
    B.m.outputs = [B.fc(B.gap(x), 10)]
    B.m.batch_size = 480
    spec = zoo.PipelineSpec("items", [det, B.m], [zoo.Edge(0, 1)], 1000.0, 540, 960, 4, 120)
    rng = np.random.default_rng(65)
    geo = octo.letterbox_geometry(540, 960, det.in_h, det.in_w)
    scenes = [synth.make_scene(rng, 4, 540, 960, counts, 16, 200, log_uniform=True) for counts in ([0, 0, 0, 0], [0, 2, 0, 1], [100] * 4, [1, 0, 2, 0])]
    batches = [([octo.to_device(v, dtype) for v in synth.planted_heads(rng, det, sc, 540, 960, geo)], [torch.from_numpy(f).cuda() for f in sc.frames]) for sc in scenes]
    got = {}
    for keep in (2, 1):
        P = octo.Pipeline(spec, keep_all_tensors=keep)
        P.set_expected_items(1, 3)
        P.set_layer_timing(True)
        got[keep], behind = [], None
        for k, (heads, frames) in enumerate(batches):
            for l, v in enumerate(heads):
                P.set_head(0, l, v)
            P.submit(frames)
            P.run()
            P.collect()
            n = len(P.get_rois(0))
            ms, kids, *_ = P.layer_info(1)
            kids = [int(k) for k in kids]
            for g in members:
                assert _launches(kids, g)[0] in ((0, 2) if keep == 2 else (0,)), kids
                assert [bool(ms[t - 1] > 0) for t in g] == [kids[t - 1] != 0 for t in g], (kids, ms)
            if keep == 2 and k in (1, 2):                # (the tiles follow the counts of the batches before: large ones go to other kernels)
                assert _launches(kids, members[0])[0] == 2, kids
            tensors = [t for g in members for t in g] + B.m.outputs
            got[keep].append([n] + [P.get_tensor(1, t, n) if n else None for t in tensors])
            after = [P.get_tensor(1, t, 3, first=60) for t in tensors]
            if behind is not None and n < 60:            # (before the large batch: whatever the memory held, NaN too)
                assert all(np.array_equal(p, q, equal_nan=True) for p, q in zip(behind, after)), k
            behind = after
        P.close()
    counts = [b[0] for b in got[1]]
    assert counts[0] == 0 and 1 <= counts[1] < 5 and counts[2] > 200 and 1 <= counts[3] < 5, counts
    for one, two in zip(got[1], got[2]):
        assert one[0] == two[0] and all(np.array_equal(p, q) for p, q in zip(one[1:], two[1:]) if p is not None)


def test_its_names():
    assert bench.conv_name(2135064032, "bf16") == "octo::conv_small_group_kernel<__bf16, 64, 32, 2, 2, 4, 1>"
    assert bench.conv_name(2136128064, "f16") == "octo::conv_small_group_kernel<_Float16, 128, 64, 4, 2, 2, 0>"
