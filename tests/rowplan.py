"""The library's rule for splitting rows (csrc/row_plan.hpp, plain host code), compiled with the host compiler: tests
state through it which launch form a shape takes."""
import ctypes
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_SRC = """
#include "row_plan.hpp"
using namespace stand;
extern "C" {
int row_parts(int64_t V, int es, int64_t rows, int K) { return plan_row_parts(V, es, rows, K); }
int commit_parts(int64_t V, int es, int64_t B, int W, int N, int R, int K) { return plan_commit_parts(V, es, B, W, N, R, K); }
int waves(int64_t rows) { return unsplit_waves(rows); }
int64_t limit(int64_t rows) { return split_limit(rows); }
int64_t vectors(int64_t V, int es) { return row_vectors(V, es); }
int whole(int64_t V, int es, int K) { return plan_row_whole(V, es, K); }
int two_parts(int64_t V, int es, int64_t rows, int K) { return plan_row_two_parts(V, es, rows, K); }
int ranges(int64_t V, int es, int64_t B) { return plan_tail_ranges(V, es, B, 16, 512); }
int two_launches(int64_t B, int64_t rows, int64_t V, int es, int K) { return plan_two_launches(B, rows, V, es, K); }
int tail_places(int64_t B, int64_t places) { return plan_tail_places(B, places); }
int tail_slots(int64_t B, int W, int groups) { return plan_tail_slots(B, W, groups); }
int tail_verify(int64_t B, int W, int groups) { return plan_tail_verify(B, W, groups); }
int tail_step(int64_t B, int W, int NO) { return plan_tail_step(B, W, NO); }
int tail_update(int W, int NO) { return plan_tail_update(W, NO); }
int loads(int verify, int all_nodes, int64_t B) { return exact_loads(verify, all_nodes, B); }
int threads() { return kPartThreads; }
int most_vectors() { return kPartVectors; }
int parts_max() { return kPartsMax; }
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
            open(src, "w").write(_SRC)
            subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                            os.path.join(ROOT, "paper_2506_04708_amd", "csrc"), "-o", so, src], check=True)
            _lib = ctypes.CDLL(so)
        i, l = ctypes.c_int, ctypes.c_int64
        _lib.row_parts.argtypes = [l, i, l, i]
        _lib.commit_parts.argtypes = [l, i, l, i, i, i, i]
        _lib.waves.argtypes = [l]
        _lib.two_launches.argtypes = [l, l, l, i, i]
        _lib.two_parts.argtypes = [l, i, l, i]
        _lib.whole.argtypes, _lib.ranges.argtypes = [l, i, i], [l, i, l]
        _lib.tail_places.argtypes = [l, l]
        _lib.tail_verify.argtypes = _lib.tail_step.argtypes = [l, i, i]
        _lib.tail_slots.argtypes = [l, i, i]
        _lib.limit.argtypes, _lib.limit.restype = [l], l
        _lib.loads.argtypes = [i, i, l]
        _lib.vectors.argtypes, _lib.vectors.restype = [l, i], l
    return _lib


def element_bytes(dtype):
    return 2 if dtype == "bf16" else 4


def row_parts(V, dtype, rows, K):
    """Parts per row of a verification; 0: not split."""
    return lib().row_parts(V, element_bytes(dtype), rows, K)


def part_registers(V, dtype, rows, K):
    """Vectors per lane of a part."""
    p = row_parts(V, dtype, rows, K)
    per = -(-lib().vectors(V, element_bytes(dtype)) // p)
    return -(-per // lib().threads())
