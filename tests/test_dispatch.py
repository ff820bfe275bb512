"""The lines between the convolution kernels, on both sides of them, by the ids that launch_conv returns (no GPU: see dispatch.py)."""
import ctypes
import math
import random

import pytest

import dispatch

SPLIT8, SPLIT4, SPLIT4_64 = 1608032032, 1604032032, 1604064032


@pytest.fixture(scope="module")
def ids(tmp_path_factory):
    exe = dispatch.program(tmp_path_factory.mktemp("dispatch"))
    return lambda layers: dispatch.kernel_ids(exe, layers)


def test_fp32_splits_of_eight_stay_splits_of_eight(ids):
    """Layers on which the two sets of estimates differ: sums of eight parts round less than those of four."""
    cases = [(14, 31, 43, 240, 16, 3, 1), (35, 12, 17, 556, 552, 3, 2), (42, 16, 13, 348, 124, 3, 1), (31, 7, 9, 152, 572, 5, 1), (118, 13, 11, 524, 40, 3, 1),
             (98, 14, 14, 84, 20, 5, 1), (19, 7, 8, 60, 472, 5, 1), (1, 112, 147, 272, 28, 3, 1), (2, 80, 119, 508, 48, 5, 1), (1, 80, 59, 680, 240, 3, 1)]
    layers = [dict(zip(("n", "h", "w", "cin", "cout", "k", "stride"), c), dtype="f32") for c in cases]
    assert ids(layers) == [SPLIT8] * len(cases)
    # and where both have four ahead, four it is
    assert ids([dict(dtype="f32", n=30, h=28, w=23, cin=104, cout=9, k=3), dict(dtype="f32", n=1, h=80, w=77, cin=68, cout=44, k=3)]) == [SPLIT4, SPLIT4_64]


SMALL, STREAM = 13, 15


def family(kid):
    return kid // 100000000


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_narrow_outputs_of_one_k_step_have_a_kernel_on_both_sides_of_every_line(ids, dtype):
    """1x1 layers of 64 channels into up to 32: conv_small_kernel below the streaming kernel's line, and where it does not take them the streaming kernel from four
    blocks of 32 pixels per compute unit on; never the general kernel in between."""
    layers, want = [], []
    for cout in (8, 24, 32):
        for place, line in ((0, 9), (1, 48)):
            for res in (0, 2):
                for blocks in (1, 3.9, 4.1, 5.9, 6.1, line - 0.1, line + 0.1):
                    h = int(blocks * 256 * 32 / 64)
                    common = dict(dtype=dtype, n=1, h=h, w=64, cin=64, cout=cout, res=res, place=place)
                    layers += [common, dict(common, upsampled=1), dict(common, n=4, split=1, hint=2)]
                    want += [SMALL if blocks < line else STREAM] + [STREAM if blocks > 4 else None] * 2
    got = ids(layers)
    assert min(got) > 0
    bad = [(l, g) for l, g, w in zip(layers, got, want) if w and family(g) != w]
    assert not bad, bad[:3]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_broken_k_steps_in_a_model_go_from_one_kernel_to_the_next(ids, dtype):
    """1x1 layers whose channels end inside a K step, into several channel tiles, in a model: conv_small_kernel up to the streaming kernel's line; conv_flow_kernel,
    which loses to both there, has none of them."""
    layers = [dict(dtype=dtype, n=1, h=int(b * 256 * 32 / ((cout + 63) // 64) / 16), w=16, cin=cin, cout=cout, res=res, place=1, second=second)
              for cin, cout in ((16, 128), (48, 96), (96, 96), (96, 192), (120, 128), (184, 320)) for b in (5, 6, 7, 8, 8.9, 9.1, 10) for res, second in ((0, 0), (2, 0), (0, 32))]
    want = [SMALL if (l["h"] * 16 + 31) // 32 * ((l["cout"] + 63) // 64) < 9 * 256 else STREAM for l in layers]
    assert [family(k) for k in ids(layers)] == want


SPLIT, PATCHES, HELD = 16, (14, 17, 18), (20,)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_split_k_is_chosen_alike_for_a_layer_of_a_model_and_a_single_call(ids, dtype):
    """Split-K adds in another order than the kernels between which the place may choose."""
    r, step = random.Random(11), 4 if dtype == "f32" else 8
    layers = []
    while len(layers) < 4000:
        k, stride = r.choice([(1, 1), (1, 1), (1, 2), (3, 1), (3, 2), (5, 2)])
        cin = r.choice([step, 64]) * r.randint(1, 32)
        cout = r.choice([8, 16, 64]) * r.randint(1, 24)
        h = r.choice([1, 7, 14, 20, 40, 57, 80, 160]) * stride
        n = max(1, int(256 * 4096 * math.exp(r.uniform(math.log(0.02), math.log(6))) / max(cout, 32) / (h // stride) ** 2))
        if k * k * cin < 60000 and 2 * n * h * h * max(cin, cout) < 1 << 30:
            layers.append(dict(dtype=dtype, n=n, h=h, w=h, cin=cin, cout=cout, k=k, stride=stride, res=r.choice([0, 0, 2]), upsampled=int(k == 1 and r.random() < 0.1),
                               split=r.choice([0, 0, max(1, n // 2)]), hint=r.choice([0, 0, max(1, n // 3)])))
    alone, place, model = ids(layers), ids([dict(l, place=1, bare=1) for l in layers]), ids([dict(l, place=1) for l in layers])
    assert sum(family(k) == SPLIT for k in alone) > 300
    differ = [(l, a, p) for l, a, p in zip(layers, alone, place) if a != p and SPLIT in (family(a), family(p))]
    assert not differ, (len(differ), differ[:2])
    # the others that differ: the lines and slices of the 3x3 kernels, else kernels of one order
    others = {family(k) for a, p in zip(alone, place) if a != p and not (family(a) in PATCHES and family(p) in PATCHES) for k in (a, p)}
    assert others <= {10, 11, 12, SMALL, STREAM}
    # and what a model keeps for conv3x3_held_kernel makes no difference but that this takes the layer
    assert all(m == p or family(m) in HELD for p, m in zip(place, model))
    assert sum(family(m) in HELD for m in model) > (25 if dtype != "f32" else -1)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_long_reductions_of_a_model_take_the_tiles_that_are_fast_there(ids, dtype):
    """1x1 layers with more K steps than the workloads have: the fastest tile by measurement, 5 % at least ahead of what constants without a cost per K step chose."""
    cases = [((1, 56, 54, 1536, 1536), 1201921288), ((11, 28, 28, 3072, 512), 1201921288), ((1, 56, 41, 4096, 2048), 1201921288),
             ((125, 20, 20, 2048, 256), 1202561288), ((125, 20, 20, 4096, 256), 1202561288)]
    assert ids([dict(zip(("n", "h", "w", "cin", "cout"), c), dtype=dtype, place=1) for c, _ in cases]) == [k for _, k in cases]


def test_every_tile_costs_something_per_k_step(tmp_path):
    """The estimates go beyond what they were fitted to: no term may be negative, and none of the two that grow with the reduction missing."""
    (tmp_path / "c.cpp").write_text('''#include "csrc/conv_small_choice.h"
template <int N> bool sound(const octo::TileCost (&t)[N]) {
  for (const auto& c : t) if (!(c.base > 0 && c.step > 0.05 && c.tile > 0 && c.latency >= 0 && c.per_mb >= 0 && c.per_operand_mb >= 0)) return false;
  return true;
}
extern "C" int both() { return sound(octo::FLOW_COST) + 2 * sound(octo::SMALL_COST); }
''')
    dispatch.compile_host(["-shared", "-fPIC", "-o", str(tmp_path / "c.so"), str(tmp_path / "c.cpp")])
    assert ctypes.CDLL(str(tmp_path / "c.so")).both() == 3


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_wide_slices_of_128_channels_end_where_a_compute_unit_has_no_place_left(ids, dtype):
    """3x3 layers of 128 channels in a model: slices of 64 channels while there are two 64 x 128 tiles per compute unit at most, whole images counted as the
    kernel cuts them, else slices of 32 (kernel ids end in the channels that two buffers hold)."""
    common = dict(dtype=dtype, cin=128, k=3, place=1, bare=1)
    cases = [(20, 40, 40, 128, 128), (21, 40, 40, 128, 64), (80, 20, 20, 128, 64), (41, 28, 28, 128, 128), (42, 28, 28, 128, 64), (2, 160, 160, 64, 128), (269, 16, 16, 64, 64),
             (48, 28, 28, 128, 64), (62, 28, 28, 128, 64), (24, 28, 28, 256, 64)]
    got = ids([dict(common, n=n, h=h, w=w, cout=co) for n, h, w, co, _ in cases])
    assert [(family(k), k % 1000) for k in got] == [(18 if co == 64 else 17, slices) for _, _, _, co, slices in cases], got
    # a count taken on the device, and single calls: slices of 32 throughout
    for change in (dict(place=0), dict(split=20, hint=20)):
        assert all(k % 1000 == 64 for k in ids([dict(common, n=n, h=h, w=w, cout=co, **change) for n, h, w, co, _ in cases[:1]]))
    # in a model it is the layers whose output channels are no multiple of 64 that come here with few tiles
    for cout, want in ((120, [(17, 128), (17, 64)]), (128, [(20, 128), (20, 128)])):
        assert [(family(k), k % 1000) for k in ids([dict(common, n=n, h=40, w=40, cout=cout, bare=0) for n in (20, 21)])] == want


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_layers_of_a_model_with_the_patch_of_the_whole_reduction_in_lds(ids, dtype):
    """conv3x3_held_kernel is asked first: where it takes a layer and who has it beyond each line - the patch kernel, split-K, conv_small_kernel, conv_flow_kernel.
    Single calls keep nothing for it."""
    cases = [(dict(n=1, h=20, cin=256, cout=256), 2014064032), (dict(n=20, h=20, cin=256, cout=256), 2014064064), (dict(n=21, h=20, cin=256, cout=256), 17),
             (dict(n=51, h=40, cin=128, cout=128), 2012064128), (dict(n=52, h=40, cin=128, cout=128), 17), (dict(n=8, h=80, cin=192, cout=192), 2012064128),
             (dict(n=9, h=80, cin=192, cout=192), 1701096064), (dict(n=5, h=80, cin=64, cout=64), 13), (dict(n=6, h=80, cin=64, cout=64), 2012064128),
             (dict(n=8, h=40, cin=256, cout=256, stride=2), 2024064064), (dict(n=16, h=40, cin=256, cout=256, stride=2), 13),
             (dict(n=300, h=14, cin=256, cout=512, stride=2, split=8, hint=111), 2024064064), (dict(n=1500, h=14, cin=256, cout=512, stride=2, split=40, hint=542), 12),
             (dict(n=900, h=28, cin=128, cout=128, split=24, hint=331), 2012064128), (dict(n=1500, h=28, cin=128, cout=128, split=40, hint=542), 17),
             (dict(n=600, h=56, cin=64, cout=64, split=16, hint=228), 18)]
    layers = [dict(l, dtype=dtype, w=l["h"], k=3) for l, _ in cases]
    got = ids([dict(l, place=1) for l in layers])
    assert [k // 10 ** (10 - len(str(w))) for k, (_, w) in zip(got, cases)] == [w for _, w in cases], got
    assert not any(family(k) in HELD for k in ids(layers))
    assert 16 in {family(k) for k in ids(layers)}                   # among them layers that are split-K's alone


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_more_than_four_slices_or_part_of_one_take_256_pixel_tiles_in_a_model_too(ids, dtype):
    """3x3 layers whose 64 x 256 tiles beat 64 x 128 ones in a model as alone; with three or four whole slices of 32 channels the place decides."""
    cases = [(35, 80, 80, 184, 128), (13, 80, 70, 184, 256), (615, 14, 12, 184, 64), (23, 80, 51, 160, 192), (157, 40, 34, 112, 128)]
    layers = [dict(zip(("n", "h", "w", "cin", "cout"), c), dtype=dtype, k=3) for c in cases]
    alone = ids(layers)
    assert ids([dict(l, place=1) for l in layers]) == alone
    assert all(k // 1000 % 10000 == 1064 for k in alone), alone                 # 256 pixels, 64 channels
    layer = dict(dtype=dtype, n=192, h=32, w=16, cin=128, cout=128, k=3)
    assert [k // 1000 % 10000 for k in ids([layer, dict(layer, place=1)])] == [1064, 64]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layer,pixels,below,beyond", [
    # (layer, output pixels per compute unit at the line, families below and beyond it)
    (dict(cin=32, cout=64, k=3, stride=2, place=1), 16 * 64, 13, 12),            # five steps across taps in a model
    (dict(cin=32, cout=64, k=3, stride=2), 1.96 * 64, 13, 12),                   # and alone
    (dict(cin=128, cout=256, k=3, stride=2), 2.75 * 16, 13, 12),
    (dict(cin=256, cout=128), 3 * 32, 13, 12),
    (dict(cin=64, cout=256), 9 * 8, 13, 15),                                     # one whole step, then resident weights
    (dict(cin=64, cout=64, k=3, place=1), 13 * 128, 1800, 1805),                 # weights in registers
    (dict(cin=64, cout=64, k=3, place=1, res=2), 10 * 128, 1800, 1805),
    (dict(cin=64, cout=64, k=3), 6 * 128, 1800, 1805),
    (dict(cin=64, cout=64, k=3), 1.96 * 64, 13, 18),                             # the patch in LDS
])
def test_both_sides_of_a_line(ids, dtype, layer, pixels, below, beyond):
    s, rows = layer.get("stride", 1), int(pixels * 256 / 32) // 8 * 8        # (the streaming kernel cuts maps into whole tiles)
    got = ids([dict(layer, dtype=dtype, n=1, h=s * (rows + d), w=s * 32) for d in (-8, 8)])
    assert [k // 10 ** (10 - len(str(want))) for k, want in zip(got, (below, beyond))] == [below, beyond], got


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_a_running_count_beyond_the_streaming_kernels_line_in_a_model(ids, dtype):
    """1x1 layers with the count on the device, the stated one between the streaming kernel's lines alone and in a model: the running count decides.  Where it is
    large they had gone to conv_flow_kernel and, one K step into more channels than that takes, to the general kernel."""
    cases = [(669, 7, 176, 232, 334), (580, 7, 96, 288, 290), (15, 57, 64, 640, 7), (71, 7, 40, 2176, 35), (28, 40, 120, 152, 14), (278, 14, 16, 80, 139)]
    layers = [dict(dtype=dtype, n=n, h=h, w=h, cin=ci, cout=co, split=split, place=1) for n, h, ci, co, split in cases]
    assert [family(k) for k in ids(layers)] == [STREAM] * len(cases)
    assert [family(k) for k in ids([dict(l, hint=l["split"] // 2) for l in layers])] == [SMALL] * len(cases)
    assert [family(k) for k in ids([dict(l, place=0) for l in layers])] == [STREAM] * len(cases)
