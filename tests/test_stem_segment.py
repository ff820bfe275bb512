"""The length of a first layer's segments (csrc/stem_segment.h, compiled for the host): as good as looking at every length, in far fewer steps."""
import ctypes
import os
import subprocess

from paper_2502_01277_amd.build import CSRC


def test_same_choice_as_every_length(tmp_path):
    (tmp_path / "s.cpp").write_text('''#include "%s/stem_segment.h"
extern "C" int segment(int h, long long strips, long long waves, int pool) { return octo::stem_segment(h, strips, waves, pool != 0); }
extern "C" int every_length(int h, long long strips, long long waves, int pool) {
  long long best = 0; int pick = 1;
  for (int seg = h; seg >= 1; --seg) {
    const long long rounds = (strips * ((h + seg - 1) / seg) + waves - 1) / waves, rows = rounds * (pool ? 2 * seg + 3 : seg + 2);
    if (seg == h || rows < best) { best = rows; pick = seg; }
  }
  return pick;
}
extern "C" int differing(int max_h, long long max_strips, long long waves) {
  int n = 0;
  for (int h = 1; h <= max_h; ++h)
    for (long long strips = 1; strips <= max_strips; strips += 1 + strips / 3)
      for (int pool = 0; pool < 2; ++pool) n += segment(h, strips, waves, pool) != every_length(h, strips, waves, pool);
  return n;
}
extern "C" double seconds(int (*f)(int, long long, long long, int), int calls) {
  timespec a, b; volatile int sink = 0;
  clock_gettime(CLOCK_PROCESS_CPUTIME_ID, &a);
  for (int i = 0; i < calls; ++i) sink = sink + f(640, 20 + i, 2048, 0);
  clock_gettime(CLOCK_PROCESS_CPUTIME_ID, &b);
  return (b.tv_sec - a.tv_sec) + 1e-9 * (b.tv_nsec - a.tv_nsec);
}
''' % CSRC)
    so = str(tmp_path / "s.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-include", "time.h", "-o", so, str(tmp_path / "s.cpp")], check=True)
    L = ctypes.CDLL(so)
    L.differing.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong]
    L.seconds.restype = ctypes.c_double
    for waves in (8, 608, 2048):
        assert L.differing(700, 60000, waves) == 0, waves
    # 640 rows: 49 lengths of 640 are looked at.  Half the time is a wide margin against the machine's moods
    fast, slow = L.seconds(L.segment, 20000), L.seconds(L.every_length, 20000)
    assert fast < 0.5 * slow, (fast, slow)
