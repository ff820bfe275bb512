"""The host side of conv3x3_held_kernel, without a GPU: the geometry of its tiles over random maps - where the loader puts every input pixel of a patch and where
a tap reads it -, and the lines of its rule on both sides."""
import ctypes as C
import random
import subprocess

import numpy as np
import pytest

import dispatch
from helpers import small_root
from paper_2502_01277_amd import binding, zoo

SOURCE = r'''
#include "csrc/conv3x3_held_choice.h"
#include <cstdio>
int main() {
  int n, h, w, ci, co, st, res, dyn, hint;
  while (scanf("%d %d %d %d %d %d %d %d %d", &n, &h, &w, &ci, &co, &st, &res, &dyn, &hint) == 9) {
    octo::ConvArgs a{};
    a.n = n; a.H = h; a.W = w; a.Cin = a.x_ld = ci; a.Cout = a.y_ld = co; a.Ho = (h - 1) / st + 1; a.Wo = (w - 1) / st + 1; a.stride_h = a.stride_w = st;
    a.kh = a.kw = 3; a.n_hint = hint; if (dyn) a.n_dyn = (int*)1; if (res) a.res = (void*)16;
    octo::HeldPlan p = octo::held_plan(st, a.W, a.Ho, a.Wo, ci, co);
    a.held = &p;
    const int can = octo::held_layer(3, 3, st, 1, h, ci, co) && octo::held_fits(a);
    printf("%d %d", can, can ? octo::held_choose(a, (long long)(dyn ? dyn : n) * a.Ho * a.Wo, 256) : -1);
    for (int i = 0; i < 3; ++i) { const octo::HeldGeom& g = p.geom[i]; printf(" %d %d %d %d %d %d %d %d", g.rows, g.TH, g.TW, g.PW, g.PH, g.halo, g.tiles_x, g.lds); }
    printf("\n");
  }
}
'''


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("held")
    (d / "held.cpp").write_text(SOURCE)
    dispatch.compile_host(["-o", str(d / "held"), str(d / "held.cpp"), "-L", dispatch.ROCM + "/lib", "-lamdhip64", "-Wl,-rpath," + dispatch.ROCM + "/lib"])

    def run(layers):
        """(n, h, w, cin, cout, stride, residual, items the count on the device is stated as (0: none there), expected): can, tile, [geometry of the three]."""
        text = "\n".join(" ".join(map(str, l)) for l in layers) + "\n"
        out = subprocess.run([str(d / "held")], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        rows = [[int(v) for v in o.split()] for o in out[:len(layers)]]
        return [(r[0], r[1], [dict(zip(("rows", "TH", "TW", "PW", "PH", "halo", "tiles_x", "lds"), r[2 + 8 * i:10 + 8 * i])) for i in range(3)]) for r in rows]
    return run


def test_every_tap_reads_the_pixel_that_the_loader_put_there(ask):
    rng = random.Random(3)
    layers = [(rng.randint(1, 9), rng.randint(4, 90), rng.randint(4, 90), 64 * rng.randint(1, 8), 64, rng.choice([1, 1, 2]), 0, 0, 0) for _ in range(300)]
    layers = [l if l[5] == 1 else (l[0], l[1] // 2 * 2) + l[2:] for l in layers]
    seen = 0
    for (n, h, w, cin, _, s, *_), (_, _, geoms) in zip(layers, ask(layers)):
        ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
        for bp, g in zip((32, 64, 128), geoms):
            if not g["rows"]:
                continue
            seen += 1
            TH, TW, PW, PH, halo, rows = (g[k] for k in ("TH", "TW", "PW", "PH", "halo", "rows"))
            assert TH * TW <= bp and 4 * wo * TH >= 3 * bp * g["tiles_x"] and TW * g["tiles_x"] >= wo
            assert PH * PW + 2 <= rows and rows % 32 == 0 and cin // 64 * rows * 128 <= g["lds"] <= 160 * 1024
            tv, tx = rng.randrange((n * ho + TH - 1) // TH), rng.randrange(g["tiles_x"])
            v0, x0 = tv * TH, tx * TW
            # the loader: row p of LDS holds input pixel (stack row, column), and its 16-byte vectors in an order that depends on a position
            holds = {}
            for p in range(rows):
                pr, pc = divmod(p, PW)
                v, x = s * v0 - 1 + pr, s * x0 - halo + pc
                if pr < PH and 0 <= v < n * h and 0 <= x < w:
                    holds[p] = (v, x, (pr * TW + pc if s == 1 else p) >> 1 & 7)
            assert not {rows - 2, rows - 1} & set(holds)
            for q in range(bp):
                ty, ox = divmod(q, TW)
                v = v0 + ty
                if ty >= TH or v >= n * ho or x0 + ox >= wo:
                    continue
                img, yy = divmod(v, ho)
                for tap in range(9):
                    r, c = tap // 3, tap % 3 - 1
                    iy, ix = s * yy + r - 1, s * (x0 + ox) + c
                    if not (0 <= iy < h and 0 <= ix < w):
                        continue
                    p = (s * ty + r) * PW + s * ox + c + halo
                    pos = p - (ty + r) * (PW - TW) if s == 1 else p
                    assert holds[p] == (img * h + iy, ix, pos >> 1 & 7)
    assert seen > 500


def test_which_layers_have_the_form(ask):
    can = [c for c, _, _ in ask([(4, 20, 20, 256, 256, 1, 0, 0, 0), (4, 20, 20, 96, 256, 1, 0, 0, 0), (4, 20, 20, 256, 255, 1, 0, 0, 0), (4, 20, 20, 576, 256, 1, 0, 0, 0),
                                 (4, 21, 20, 256, 256, 2, 0, 0, 0), (4, 20, 21, 256, 256, 2, 0, 0, 0)])]
    assert can == [1, 0, 0, 0, 0, 1]


def test_both_sides_of_the_lines(ask):
    cases = [
        ((4, 20, 20, 256, 256, 1, 0, 0, 0), 0), ((8, 20, 20, 256, 256, 1, 0, 0, 0), 1), ((16, 20, 20, 256, 256, 1, 0, 0, 0), 2),
        ((32, 20, 20, 256, 256, 1, 0, 0, 0), -1),                                       # more than are resident
        ((63, 7, 7, 512, 512, 1, 0, 0, 0), 2), ((134, 7, 7, 512, 512, 1, 0, 0, 0), -1),
        ((48, 40, 40, 128, 128, 1, 0, 0, 0), 2), ((52, 40, 40, 128, 128, 1, 0, 0, 0), -1), ((64, 40, 40, 128, 128, 1, 0, 0, 0), -1),      # five per compute unit
        ((8, 80, 80, 192, 192, 1, 0, 0, 0), 2), ((9, 80, 80, 192, 192, 1, 0, 0, 0), -1), ((10, 80, 80, 192, 192, 1, 0, 0, 0), -1),
        ((480, 40, 40, 128, 128, 1, 0, 48, 48), -1), ((480, 40, 40, 128, 128, 1, 0, 12, 12), 2), ((480, 14, 14, 256, 256, 1, 0, 41, 41), 2),
        ((5, 80, 80, 64, 64, 1, 0, 0, 0), -1), ((6, 80, 80, 64, 64, 1, 0, 0, 0), 2), ((12, 80, 80, 64, 64, 1, 0, 0, 0), -1),
        ((2, 80, 80, 128, 128, 2, 0, 0, 0), 0), ((6, 80, 80, 128, 128, 2, 0, 0, 0), -1), ((1, 14, 14, 128, 256, 2, 0, 0, 0), -1), ((1, 160, 160, 64, 128, 2, 0, 0, 0), -1),
        ((30, 14, 14, 256, 512, 2, 0, 0, 0), 1), ((134, 14, 14, 256, 512, 2, 0, 0, 0), -1),
        # 64 x 32 and 64 x 64 tiles by the running count; what else is decided by the stated one
        ((480, 14, 14, 256, 256, 1, 0, 4, 4), 0), ((480, 14, 14, 256, 256, 1, 0, 4, 300), 1), ((480, 14, 14, 256, 256, 1, 0, 41, 3), 2),
        ((480, 14, 14, 256, 256, 1, 0, 200, 3), -1)]
    assert [t for _, t, _ in ask([c for c, _ in cases])] == [t for _, t in cases]


def test_a_count_on_the_device_may_be_many_times_the_stated_one(ask):
    """(Stated count, capacity, map, channels, stride): layers of downstream classifiers whose running count may be many times the stated one, on both sides of the lines."""
    cases = [
        ((40, 1500, 14, 256, 512, 2), False), ((24, 900, 14, 256, 512, 2), False), ((8, 300, 14, 256, 512, 2), True),          # 65 : 104 us, 50 : 62, 38 : 23
        ((32, 1200, 8, 512, 512, 2), True), ((72, 2700, 8, 512, 512, 2), False), ((128, 4800, 8, 128, 256, 2), False),
        ((16, 600, 56, 64, 64, 1), False), ((32, 1200, 56, 64, 64, 1), False),                                                   # 67 : 73
        ((24, 900, 28, 128, 128, 1), True), ((32, 1200, 28, 128, 128, 1), False), ((40, 1500, 28, 128, 128, 1), False),         # 79 : 81, 98 : 106, 113 : 135
        ((48, 1800, 14, 256, 256, 1), True), ((64, 2400, 14, 256, 256, 1), False), ((64, 2048, 14, 256, 256, 1), True),         # 132 : 133, 172 : 180; no room for more than 32 times
        ((64, 2400, 7, 512, 512, 1), True), ((72, 2700, 7, 512, 512, 1), False), ((80, 2560, 7, 512, 512, 1), True), ((80, 2561, 7, 512, 512, 1), False),      # 217 : 183, 215 : 228
        # no room for more than eight times the stated count: as with a count that the host knows
        ((64, 512, 8, 128, 256, 2), True), ((64, 513, 8, 128, 256, 2), False), ((32, 256, 28, 128, 128, 1), True), ((32, 257, 28, 128, 128, 1), False),
        ((16, 128, 56, 64, 64, 1), True), ((16, 129, 56, 64, 64, 1), False)]
    got = ask([(cap, hw, hw, ci, co, s, 0, stated, h) for (stated, cap, hw, ci, co, s), _ in cases for h in (0, min(cap, 14 * stated))])
    taken = [t >= 0 for _, t, _ in got]
    assert taken[::2] == taken[1::2]                       # a matter of the stated count alone
    assert taken[::2] == [w for _, w in cases]
    # the same layers with a count that the host knows
    known = [t >= 0 for _, t, _ in ask([(stated, hw, hw, ci, co, s, 0, 0, 0) for (stated, _, hw, ci, co, s), _ in cases])]
    assert known.count(True) > taken[::2].count(True)


def test_no_hole_between_the_lines(ask):
    """Once a batch has outgrown the kernel, no larger one takes it again."""
    for h, ci, top in ((40, 128, 51), (80, 192, 8), (20, 256, 20), (40, 384, 3)):
        taken = [t >= 0 for _, t, _ in ask([(n, h, h, ci, ci, 1, 0, 0, 0) for n in range(1, 80)])]
        assert taken.index(False) == top and not any(taken[top:]), (h, ci, taken.index(False))


@pytest.mark.parametrize("stride,cin,cout,h,kept", [(2, 64, 128, 40, False), (1, 64, 128, 40, True), (2, 128, 128, 40, True), (1, 64, 64, 3, False), (1, 512, 64, 131, True), (2, 512, 64, 20, True)])
def test_weights_are_kept_twice_only_where_a_launch_can_read_them(ask, stride, cin, cout, h, kept):
    """A model's device memory with a layer of padding 1 against the same of padding 0, which has smaller tensors and is never kept twice."""
    size = []
    for pad in (0, 1):
        B = zoo._Builder("t", "bf16", h, h, "classifier", np.random.default_rng(1))
        B.ch = [cin]
        B.m.in_c = cin
        B.m.outputs = [B.fc(B.gap(B.conv(0, cout, 3, stride, p=pad)), 8)]
        B.m.batch_size = 1
        keep, n = [], C.c_size_t()
        d = binding.pipeline_desc(zoo.PipelineSpec("t", [small_root("bf16"), B.m], [], 200.0, 32, 32, 1, 1), keep)
        assert binding.lib().octo_pipeline_workspace_size(C.byref(d), C.byref(n)) == binding.OK
        size.append(n.value)
    copy, tensors = 18 * cin * cout, 2 * cout * (((h - 1) // stride + 1) ** 2 - ((h - 3) // stride + 1) ** 2)
    assert tensors + 1024 < copy and (size[1] - size[0] >= copy) == kept and size[1] - size[0] <= copy * kept + tensors + 1024
    # and no launch of a layer without the copy would be taken
    taken = any(t >= 0 for _, t, _ in ask([(n, h, h, cin, cout, stride, 0, 0, 0) for n in range(1, 200)]))
    assert taken == kept
