"""The library's dispatch rules (csrc/dispatch_rules.h) and the walk of a wave over its tiles (csrc/tile_walk.h), compiled
for the host: a test that sits where a rule changes its answer asks the rule itself."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_28458_amd", "csrc")

_SHIM = """
#include "dispatch_rules.h"
#include "tile_walk.h"
extern "C" int in_ring(long T, long s_max, long packed, long fp8, long without, long with) {
  return hisa::hist_in_ring(T, s_max, packed, fp8, without, with);
}
extern "C" int key_ranges(long q_groups, long first, long last) { return hisa::prefill_split(q_groups, first, last); }
extern "C" int tile_of_walk(long j, long nj, long j0, long wave, long n_waves) {
  return hisa::walk_tile(j, nj, j0, wave, n_waves);
}
extern "C" int f32_one_launch(long T, long n, long H, long d) { return hisa::rows_f32_one_launch(T, n, H, d); }
extern "C" int f32_waves(long T, long n) { return hisa::rows_f32_waves(T, n); }
extern "C" int in_step(long n_tiles, long n_waves) { return hisa::walk_in_step(n_tiles, n_waves); }
extern "C" int start_of_walk(long n_tiles, long n_waves, long now, long ticks) {
  return hisa::walk_start(n_tiles, n_waves, (uint32_t)now, ticks);
}
extern "C" int ticks_of_walk(long key_bytes, long fp8) { return hisa::walk_ticks(key_bytes, fp8); }
extern "C" int one_launch(long T, long M, long H) { return hisa::stage1_one_launch(T, M, H); }
extern "C" int tiles_per_wave(long T, long n_tiles) { return hisa::gather_tiles_per_wave(T, n_tiles); }
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
        with open(src, "w") as f:
            f.write(_SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so], check=True)
        return ctypes.CDLL(so)


def _call(name, *args):
    fn = getattr(_lib(), name)
    fn.argtypes, fn.restype = [ctypes.c_long] * len(args), ctypes.c_int
    return fn(*args)


def tiles_per_wave(T, n_tiles):
    return _call("tiles_per_wave", T, n_tiles)


def in_ring(T, s_max, packed, fp8, without, with_):
    return bool(_call("in_ring", T, s_max, packed, fp8, without, with_))


def key_ranges(T, rows_first, rows_last):
    return _call("key_ranges", -(-T // 8), rows_first, rows_last)


def tile_of_walk(j, nj, j0, wave, n_waves):
    return _call("tile_of_walk", j, nj, j0, wave, n_waves)


def f32_one_launch(T, n, H, d):
    return bool(_call("f32_one_launch", T, n, H, d))


def f32_waves(T, n):
    return _call("f32_waves", T, n)


def walk_start(n_tiles, n_waves, now, ticks):
    """First tile of the walks, as the kernel has it: 0 unless they may begin elsewhere."""
    return _call("start_of_walk", n_tiles, n_waves, now, ticks) if _call("in_step", n_tiles, n_waves) else 0


def walk_ticks(key_bytes, fp8):
    return _call("ticks_of_walk", key_bytes, fp8)


def stage1_one_launch(T, M, H):
    return bool(_call("one_launch", T, M, H))
