"""The check of pivots behind an elimination (csrc/pivot.hpp), compiled for the host: it never passes a pivot at or below its threshold."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_03423_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("pivot")
    (d / "p.cpp").write_text('#include "pivot.hpp"\nextern "C" void check(const double *r, const double *thr, int n, unsigned char *out) {\n'
                             '  for (int i = 0; i < n; ++i) out[i] = rsvd::pivot_surely_above(r[i], thr[i]);\n}\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-I", CSRC, str(d / "p.cpp"), "-o", str(d / "p.so")], check=True)
    fn = C.CDLL(str(d / "p.so")).check

    def run(r, thr):
        r, thr, out = np.ascontiguousarray(r), np.ascontiguousarray(thr), np.zeros(len(r), np.uint8)
        fn(r.ctypes.data_as(C.c_void_p), thr.ctypes.data_as(C.c_void_p), len(r), out.ctypes.data_as(C.c_void_p))
        return out.astype(bool)
    return run


def _ulps(x, k):
    return (np.asarray(x, np.float64).view(np.int64) + k).view(np.float64)        # (positive values)


@pytest.mark.parametrize("scale", [1e-300, 1e-160, 1e-12, 1.0, 1e100])
def test_pivots_next_to_the_threshold(check, scale):
    thr = np.concatenate([scale * np.exp(np.random.default_rng(1).uniform(-3, 3, 4000)), scale * 2.0 ** -np.arange(8.0)])
    for below in range(4):                                  # pivots at the threshold and up to three ulp below it
        for off in (-2, -1, 0, 1, 2):                       # their roots, off by as much as the kernel's may be
            assert not check(_ulps(np.sqrt(_ulps(thr, -below)), off), thr).any()
    for off in (-2, -1, 0, 1, 2):                           # and well above: no second elimination for nothing
        assert check(_ulps(np.sqrt(thr * (1 + 1e-14)), off), thr).all()


def test_what_is_no_pivot(check):
    bad = np.array([np.nan, 0.0, 5e-162])
    assert not check(bad, np.full(3, 1e-300)).any() and not check(np.full(3, np.nan), np.array([0.0, 1.0, np.inf])).any()
    assert not check(np.array([0.0]), np.array([0.0])).any()
