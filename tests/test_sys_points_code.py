"""The points of SysPoints (csrc/dpf_seg.hpp), which the filters resample by, are
the bits of sys_point, the rule of the primitives and of the oracle: both compiled
for the host from the header's own text (IEEE double arithmetic on either side; the
GPU's power-of-two scaling is ldexp) and compared over every count that the classes
hold, totals from one weight to all, and offsets next to both ends."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

SEG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1203_2394_amd", "csrc",
                   "dpf_seg.hpp")


def _definition(text, start):
    """The definition beginning with `start`, to its closing brace."""
    i = text.index(start)
    depth, j = 0, text.index("{", i)
    for k in range(j, len(text)):
        depth += {"{": 1, "}": -1}.get(text[k], 0)
        if depth == 0:
            return text[i:k + 1]
    raise AssertionError("unbalanced definition")


@pytest.fixture(scope="module")
def points(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    text = re.sub(r"//[^\n]*", "", open(SEG).read())
    src = "\n".join(["#include <cmath>", "#define __device__", "#define __forceinline__ inline",
                     "#define __builtin_amdgcn_ldexp std::ldexp",
                     _definition(text, "__device__ __forceinline__ double sys_point("),
                     _definition(text, "struct SysPoints") + ";",
                     'extern "C" long both(int n, long m, const double* u, const double* total, const int* k, long* at) {',
                     "  long bad = 0;",
                     "  for (long i = 0; i < m; ++i) {",
                     "    const SysPoints p(u[i], total[i], n);",
                     "    const double a = p(k[i]), b = sys_point(k[i], u[i], total[i], n);",
                     "    if (!(a == b)) { if (!bad) *at = i; ++bad; }",
                     "  }",
                     "  return bad;",
                     "}"])
    d = tmp_path_factory.mktemp("sys_points")
    (d / "p.cpp").write_text(src)
    subprocess.run([cxx, "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-o", str(d / "p.so"), str(d / "p.cpp")],
                   check=True)
    L = ctypes.CDLL(str(d / "p.so"))
    L.both.restype = ctypes.c_long
    return L.both


def _ptr(a, ty):
    return np.ascontiguousarray(a).ctypes.data_as(ctypes.POINTER(ty))


def test_points_are_the_primitives_points(points):
    g = np.random.default_rng(6)
    for n in range(1, 4097):
        k = np.concatenate([np.arange(min(n, 40)), g.integers(0, n, size=120), [n - 1] * 20]).astype(np.int32)
        m = k.size
        u = (2.0 * g.integers(0, 1 << 52, size=m) + 1.0) * 2.0 ** -53
        u[:6] = [2.0 ** -53, 1.0 - 2.0 ** -53, 0.5, np.nextafter(0.5, 0), 2.0 ** -53, 1.0 - 2.0 ** -53]
        # sums of up to n weights of at most 1: one weight, all equal, anything between
        total = 1.0 + g.random(m) * (n - 1)
        total[::5] = 1.0
        total[1::5] = n
        total[2::9] = np.nextafter(total[2::9], 1e9)
        at = ctypes.c_long(-1)
        u, total, k = map(np.ascontiguousarray, (u, total, k))
        bad = points(n, ctypes.c_long(m), _ptr(u, ctypes.c_double), _ptr(total, ctypes.c_double), _ptr(k, ctypes.c_int),
                     ctypes.byref(at))
        assert bad == 0, (n, bad, int(k[at.value]), float(u[at.value]).hex(), float(total[at.value]).hex())
