"""The library's rules on sizes (csrc/rules.hpp), compiled for the host: tests
choose and check the pools that are to reach a kernel by the rule itself, not by
a copy of it."""
import ctypes
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2609_36830_amd", "csrc", "rules.hpp")
SOURCE = """
#include "%s"
using namespace pace;
extern "C" {
int by_traj(int64_t n, int64_t nt) { return score_by_traj(n, nt); }
int waves(int64_t n, int64_t nt) { return traj_waves(n, nt); }
int64_t cap(int64_t n, int64_t nt) { return score_traj_cap(n, nt); }
int narrow(int64_t n, int64_t nt, int32_t v) { return score_traj_narrow(n, nt, v); }
int mode(int32_t v) { return reduce_mode(v); }
int in_rank(int64_t n, int64_t ng) { return group_means_in_rank(n, ng); }
int small(int64_t n, int64_t nt, int cols, int64_t b) { return small_step_ok(n, nt, cols, b); }
}
""" % HEADER
PACKED, NARROW, WIDE = 0, 1, 2


def _load():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as fh:
            fh.write(SOURCE)
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", src, "-o", so])
        L = ctypes.CDLL(so)
    i32, i64 = ctypes.c_int32, ctypes.c_int64
    for name, res, args in (("by_traj", i32, (i64, i64)), ("waves", i32, (i64, i64)), ("cap", i64, (i64, i64)),
                            ("narrow", i32, (i64, i64, i32)), ("mode", i32, (i32,)), ("in_rank", i32, (i64, i64)),
                            ("small", i32, (i64, i64, i32, i64))):
        f = getattr(L, name)
        f.restype, f.argtypes = res, args
    return L


_lib = None


def rules():
    global _lib
    if _lib is None:
        _lib = _load()
    return _lib
