"""bench.py names the convolution kernels by the id that a launch returns.  Every instance that a launcher of the sources can start is
taken through the id functions the launchers use (csrc/kernel_ids.h, compiled for the host) and back to its name."""
import ctypes
import os
import re
import subprocess

import pytest

import bench
from paper_2502_01277_amd.build import CSRC

CTYPE = {"f16": "_Float16", "bf16": "__bf16", "f32": "float", "f8": "octo::f8"}


@pytest.fixture(scope="module")
def ids(tmp_path_factory):
    d = tmp_path_factory.mktemp("kernel_ids")
    fns = {"conv_kernel_id": 7, "mid_kernel_id": 7, "stream3_kernel_id": 4, "stream1_kernel_id": 2, "ksplit_kernel_id": 3, "stem_kernel_id": 4}
    src = '#include "%s/kernel_ids.h"\n' % CSRC
    for f, n in fns.items():
        names = ["a%d" % i for i in range(n)]
        src += 'extern "C" int %s(%s) { return octo::%s(%s); }\n' % (f, ", ".join("int " + a for a in names), f, ", ".join(names))
    (d / "ids.cpp").write_text(src)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", str(d / "ids.so"), str(d / "ids.cpp")], check=True)
    return ctypes.CDLL(str(d / "ids.so"))


def instances(launcher, *files):
    """Template arguments of every call of a launcher: ('T' or a type, [numbers])."""
    found = set()
    for f in files:
        text = open(os.path.join(CSRC, f)).read()
        for m in re.finditer(r"\b%s<(T|f8), ([^>]*)>\(" % launcher, text):
            found.add((m.group(1), tuple({"true": 1, "false": 0}.get(v) if v in ("true", "false") else int(v) for v in m.group(2).split(", "))))
    assert found, launcher
    return sorted(found)


def types(t):
    return ["f16", "bf16"] if t == "T" else ["f8"]


def test_3x3_patch_kernels(ids):
    for t, (bc, bp, wc, kv, nst, maxp, minb) in instances("launch_mid_cfg", "conv3x3_mid.h", "conv.hip"):
        vn = 8 if t == "T" else 16
        for dt in types(t):
            for cin in (kv * vn, kv * vn + 8):
                for cout in (24, 200):
                    kid = ids.mid_kernel_id(bc, bp, kv, vn, maxp, cin, cout)
                    assert bench.conv_name(kid, dt) == "octo::conv3x3_mid_kernel<%s, %d, %d, %d, %d, %d, %d, %d>" % (CTYPE[dt], bc, bp, wc, kv, nst, maxp, minb)
    for _, args in instances("launch_stream3_cfg", "conv3x3_stream.h"):
        for dt in types("T"):
            for cin in (args[1] * 16, args[1] * 16 - 8):
                kid = ids.stream3_kernel_id(args[0], args[1], args[2], cin)
                assert bench.conv_name(kid, dt) == "octo::conv3x3_stream_kernel<%s, %s>" % (CTYPE[dt], ", ".join(map(str, args)))


def test_1x1_split_k_and_first_layer_kernels(ids):
    for _, (tc,) in instances("launch_stream_cfg", "conv1x1.hip"):
        for cin in (16, 192):
            assert bench.conv_name(ids.stream1_kernel_id(tc, cin), "bf16") == "octo::conv1x1_stream_kernel<__bf16, %d>" % tc
    for _, (tc, tp, nw, ks) in instances("launch_ksplit_cfg", "conv_ksplit.h"):
        for dt in CTYPE:
            kid = ids.ksplit_kernel_id(32 * tc, 32 * tp * (nw // ks), ks)
            assert bench.conv_name(kid, dt) == "octo::conv_ksplit_kernel<%s, %d, %d, %d, %d>" % (CTYPE[dt], tc, tp, nw, ks)
    for _, (bc, kh, pkw, pool) in instances("launch_stem_cfg", "stem.hip"):
        kid = ids.stem_kernel_id(bc, kh, pkw, pool)
        assert bench.conv_name(kid, "f16") == "octo::stem_conv_kernel<_Float16, %d, %d, %d, %s>" % (bc, kh, pkw, "true" if pool else "false")


def test_general_kernel(ids):
    for t, a in instances("launch_cfg", "conv.hip"):
        a = a + (0,) * (10 - len(a))
        for dt in ["f32", "f16", "bf16"] if t == "T" else ["f8"]:
            kid = ids.conv_kernel_id(a[0], a[1], a[4], a[6], *a[7:])
            assert bench.conv_name(kid, dt) == "octo::conv_mfma_kernel<%s, %s, %s>" % (
                CTYPE[dt], ", ".join(map(str, a[:7])), ", ".join("true" if v else "false" for v in a[7:]))


def test_kernels_whose_loads_run_across_tiles(tmp_path):
    src = '#include "%s/kernel_ids.h"\nextern "C" int flow_kernel_id(int a, int b, int c, int d) { return octo::flow_kernel_id(a, b, c, d); }\n' % CSRC
    (tmp_path / "ids.cpp").write_text(src)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", str(tmp_path / "ids.so"), str(tmp_path / "ids.cpp")], check=True)
    fn = ctypes.CDLL(str(tmp_path / "ids.so")).flow_kernel_id
    for _, (nt, bc, bp, wc, kv, nst, minb) in instances("launch_flow_cfg", "conv_flow.h"):
        for mode in range(3):
            assert bench.conv_name(fn(bc, bp, kv, mode), "bf16") == "octo::conv_flow_kernel<__bf16, %d, %d, %d, %d, %d, %d, %d, %d>" % (nt, bc, bp, wc, kv, nst, minb, mode)


def test_kernels_for_launches_of_few_tiles(tmp_path):
    src = '#include "%s/kernel_ids.h"\nextern "C" int small_kernel_id(int a, int b, int c, int d) { return octo::small_kernel_id(a, b, c, d); }\n' % CSRC
    (tmp_path / "ids.cpp").write_text(src)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", str(tmp_path / "ids.so"), str(tmp_path / "ids.cpp")], check=True)
    fn = ctypes.CDLL(str(tmp_path / "ids.so")).small_kernel_id
    found = instances("launch_small_cfg", "conv_small.h")
    assert {(bc, bp) for _, (bc, bp, *_) in found} == set(bench.SMALL)
    for _, (bc, bp, wc, wp, minb) in found:
        # fp32 has two ways to make addresses more, and no 128 x 64 tiles
        for dt, modes in (("f16", 3), ("bf16", 3), ("f32", 5 if bc < 128 else 0)):
            for mode in range(modes):
                assert bench.conv_name(fn(bc, bp, wc, mode), dt) == "octo::conv_small_kernel<%s, %d, %d, %d, %d, %d, %d>" % (CTYPE[dt], bc, bp, wc, wp, minb, mode)


def test_an_unknown_id_has_a_name_too():
    for kid in (1403064128 + 4000000, 1804064128, 1700064999, 1899999999, 1499999999, 1805128128):
        for dt in CTYPE:
            assert "conv" in bench.conv_name(kid, dt)
