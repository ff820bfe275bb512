"""Convolutions that do not depend on one another in one launch (conv_small_group_kernel): a shortcut beside its block's first layer, and three 1x1 layers of different inputs and
channel counts.  Every tensor bit for bit what the layers give in launches of their own, with buffers that are kept and with buffers that are reused."""
import numpy as np
import pytest

from oracle import nn
from paper_2502_01277_amd import zoo
from helpers import TOL, rel_err, small_root


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


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("make,n,h,w", [(_shortcut, 1, 9, 11), (_shortcut, 11, 28, 28), (_shortcut, 40, 41, 39), (_heads, 1, 5, 3), (_heads, 3, 20, 21), (_heads, 9, 40, 40)])
def test_bit_for_bit_what_the_layers_give_alone(octo, dtype, make, n, h, w):
    m, groups = make(dtype, n, h, w)
    x = zoo.round_to_dtype(np.random.default_rng(63).uniform(-1, 1, (n, h, w, 16)).astype(np.float32), dtype)
    members = [t for g in groups for t in g]
    got, kids = {}, {}
    for keep in (1, 2, 0):
        P = octo.Pipeline(zoo.PipelineSpec("t", [small_root(dtype), m], [], 200.0, 32, 32, 1, 1), keep_all_tensors=keep)
        for _ in range(2):                               # buffers hold the results of an earlier run
            P.run_model_on(1, octo.to_device(x, dtype))
        got[keep] = {t: P.get_tensor(1, t, n) for t in (members if keep else []) + [m.outputs[0]]}
        kids[keep] = [int(q) for q in P.layer_info(1)[1]]
        P.close()
    ref = nn.run_model(m, x[:1], keep_all=True)
    for t in members:
        assert rel_err(got[2][t][:1], ref[t]) <= TOL[dtype], t
        assert np.array_equal(got[2][t], got[1][t]), t
    assert np.array_equal(got[0][m.outputs[0]], got[1][m.outputs[0]])
    # members that conv_small_kernel takes have one tile
    for g in groups:
        tiles = {kids[2][t - 1] for t in g if kids[2][t - 1] // 100000000 == 13}
        assert len(tiles) <= 1, kids[2]
    if n < 40:
        assert sum(kids[2][t - 1] // 100000000 == 13 for t in groups[0]) == len(groups[0]), kids[2]
