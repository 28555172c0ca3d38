"""csrc/cada_rows_split.h for tests: compiled with the host compiler, called through ctypes."""
import ctypes as C
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (p, M, B, rule) whose rows are cut evenly, so that shares meet several workers: five, six and seven quads per lane
SHARED_WORKERS = [(8196, 129, 19, 2), (8199, 137, 21, 1), (8193, 600, 2, 2), (10240, 129, 20, 3), (10241, 131, 19, 1), (12288, 133, 20, 2),
                  (12289, 129, 19, 1), (14335, 129, 19, 2), (14336, 300, 1, 1)]

_SRC = """
#include "cada_rows_split.h"
using namespace cada;
extern "C" {
void split(int M, int B, long p, int *out) { const WideSplit w = wide_split(M, B, p); out[0] = w.shares; out[1] = w.rows; out[2] = w.per; out[3] = wide_slots(w); }
int preferred(int M, int B, long p, int vec) { return rows_preferred(M, B, p, vec); }
void narrow(int M, int B, long p, int *out) { const RowsSplit r = rows_split(M, B, p); out[0] = r.shares; out[1] = r.rows; }
int first(const WideSplit *w, int c) { return wide_first(*w, c); }
int share(const WideSplit *w, int f) { return wide_share(*w, f); }
int slot(const WideSplit *w, int c, int m) { return wide_slot(*w, c, m); }
}
"""


class _W(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("M", "B", "shares", "rows", "per")]


def compile_split(tmp):
    src, lib = os.path.join(str(tmp), "split.cc"), os.path.join(str(tmp), "split.so")
    with open(src, "w") as f:
        f.write(_SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2012_15469_amd", "csrc"), "-o", lib, src], check=True)
    dll = C.CDLL(lib)

    class Split:
        def __init__(self, M, B, p):
            out = (C.c_int * 4)()
            dll.split(M, B, C.c_long(p), out)
            self.shares, self.rows, self.per, self.slots = out
            self._w = _W(M, B, self.shares, self.rows, self.per)

        def first(self, c): return dll.first(C.byref(self._w), c)
        def share(self, f): return dll.share(C.byref(self._w), f)
        def slot(self, c, m): return dll.slot(C.byref(self._w), c, m)

    def narrow(M, B, p):
        out = (C.c_int * 2)()
        dll.narrow(M, B, C.c_long(p), out)
        return tuple(out)

    Split.narrow = staticmethod(narrow)
    Split.preferred = staticmethod(lambda M, B, p, vec: bool(dll.preferred(M, B, C.c_long(p), vec)))
    return Split
