"""The rules that run in the kernels (csrc/rules.h, compiled for the CPU)
against their restatements in Python, which the other tests compare with the
bisection tree and with exact quotients."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from test_edge_levels import EDGES, LEVELS
from test_exit_face_rule import directions, dots
from test_locate_rule import S, fold, roots_of

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_11510_amd", "csrc")
SHIM = """
#include "rules.h"
extern "C" {
uint32_t edges_upto(int d, int smax) { return tv::edges_upto(d, smax); }
uint64_t fold_below(double a, double b, double c, double s, int dmax, uint64_t h) { return tv::fold_path<false>(a, b, c, s, dmax, h); }
uint64_t fold_above(int32_t a, int32_t b, int32_t c, int32_t s, int dmax, uint64_t h) { return tv::fold_path<true>(a, b, c, s, dmax, h); }
void seg_dirs(const float* d, long n, float* r, float* dot) {
  for (long i = 0; i < n; i++) {
    tv::SegDirs s;
    tv::seg_dirs(d[3 * i], d[3 * i + 1], d[3 * i + 2], s);
    for (int k = 0; k < 9; k++) r[9 * i + k] = s.r[k], dot[9 * i + k] = s.d[k];
  }
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-D__host__=", "-D__device__=", "-shared", "-fPIC", "-I", CSRC,
                    "-o", str(d / "rules.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "rules.so"))
    lib.edges_upto.restype = ctypes.c_uint32
    lib.fold_below.restype = lib.fold_above.restype = ctypes.c_uint64
    return lib


def test_edges(rules):
    for d in range(61):
        for smax in range(-1, 61):
            want = sum(1 << k for k, e in enumerate(EDGES) if d + LEVELS[3 - d % 3][e] <= smax)
            assert rules.edges_upto(d, smax) == want, (d, smax)


def test_folds(rules):
    rng = np.random.default_rng(3)
    pts = [rng.integers(0, 9, 3) / 8 for _ in range(100)] + [rng.random(3).astype(np.float32).astype(float) for _ in range(300)]
    for p in pts:
        for r, f in roots_of([float(x) * S for x in p]):
            for d in (0, 1, 2, 3, 24, 56, 57, 60):
                got = rules.fold_below(*(ctypes.c_double(x) for x in (*f, S)), d, ctypes.c_uint64(8 + r))
                assert got == fold(*f, float(S), d, 8 + r, False)
    # the links' points: 8 x (3 x a face's centroid) plus its normal, in units of 1/24
    for _ in range(400):
        q = 8 * rng.integers(0, 3 * S + 1, 3) + rng.integers(-1, 2, 3)
        q = [int(x) for x in np.clip(q, 0, 24 * S)]
        for r, f in roots_of(q):
            for d in (1, 9, 24, 56, 60):
                got = rules.fold_above(*(ctypes.c_int32(x) for x in (*f, 24 * S)), d, ctypes.c_uint64(8 + r))
                assert got == fold(*f, 24 * S, d, 8 + r, True)


@pytest.mark.parametrize("kind", ["random", "axes", "diagonals", "grazing", "tiny"])
def test_reciprocals(rules, kind):
    d = np.ascontiguousarray(directions(kind, 20000, np.random.default_rng(4)))
    d[:3] = [[0, 0, 0], [np.nan, 1, 0], [-0.0, 1, 0]]
    r, dot = np.empty((len(d), 9), np.float32), np.empty((len(d), 9), np.float32)
    rules.seg_dirs(*(a.ctypes.data_as(ctypes.c_void_p) for a in (d,)), ctypes.c_long(len(d)),
                   *(a.ctypes.data_as(ctypes.c_void_p) for a in (r, dot)))
    want = dots(d)
    assert np.array_equal(dot, want, equal_nan=True)
    tiny = (d == 0).all(axis=1) | ((want != 0) & ~((want <= -np.float32(2.0 ** -40)) | (want >= np.float32(2.0 ** -40)))).any(axis=1)
    with np.errstate(all="ignore"):
        rec = np.where(tiny[:, None], np.float32(0), np.where(want == 0, np.float32(np.nan), np.float32(1) / want))
    assert np.array_equal(r, rec.astype(np.float32), equal_nan=True)
