"""CPU checks of the filter pass's test of the bounds (csrc/reach.hpp, compiled for the host): what it lists and what it
must never list, for rows past the last source, zero sources, zero keys and keys with infinities."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2509_00388_amd import build

CODE = r"""
#include <cmath>
#define __device__
#define __forceinline__ inline
#include "reach.hpp"
extern "C" uint32_t hits(const float *bound, const float *inv, const int *there, const float *dot, float norm)
{
    float det[16];
    for (int i = 0; i < 16; ++i) det[i] = gkv::dot_bound(bound[i], inv[i], there[i] != 0);
    uint32_t misses = 0;
    for (int v = 3; v >= 0; --v) {
        const float d4[4] = {dot[4 * v], dot[4 * v + 1], dot[4 * v + 2], dot[4 * v + 3]};
        const float t4[4] = {det[4 * v], det[4 * v + 1], det[4 * v + 2], det[4 * v + 3]};
        misses = gkv::push_misses(misses, d4, t4, gkv::norm_for_test(norm));
    }
    return ~misses & 0xffffu;
}
"""
NAN = np.array([0x7FC00000, 0xFFC00000], dtype=np.uint32).view(np.float32)   # of either sign


@pytest.fixture(scope="module")
def hits(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    where = tmp_path_factory.mktemp("reach")
    (where / "reach.cpp").write_text(CODE)
    lib = where / "reach.so"
    subprocess.run([cxx, "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I", build.CSRC, "-o", str(lib),
                    str(where / "reach.cpp")], check=True)
    fn = ctypes.CDLL(str(lib)).hits
    fn.restype = ctypes.c_uint32

    def call(bound, inv, there, dot, norm):
        f = [np.broadcast_to(np.asarray(a, dtype=np.float32), 16).copy() for a in (bound, inv, dot)]
        t = np.broadcast_to(np.asarray(there, dtype=np.int32), 16).copy()
        ptr = [ctypes.c_void_p(a.ctypes.data) for a in (f[0], f[1], t, f[2])]
        bits = fn(*ptr, ctypes.c_float(float(norm)))
        return [(bits >> i) & 1 for i in range(16)]

    return call


NORMS = [0.0, 1e-20, 1.0, 11.0, 1e18, np.inf, float(NAN[0]), float(NAN[1])]
DOTS = [0.0, -0.0, 1.0, -1.0, 3e38, np.inf, -np.inf, float(NAN[0]), float(NAN[1])]


@pytest.mark.parametrize("norm", NORMS)
@pytest.mark.parametrize("dot", DOTS)
def test_rows_past_the_last_source_are_never_listed(hits, norm, dot):
    """Their list would be the next head's.  One source of the sixteen is there, and its dot reaches what it can."""
    for bound in (-np.inf, -0.5, 0.0, 0.5, 1.0):
        for inv in (0.0, 0.1):
            got = hits(bound, inv, [1] + [0] * 15, [0.0] + [dot] * 15, norm)
            assert not any(got[1:]), (bound, inv, norm, dot)


@pytest.mark.parametrize("norm", [0.0, 1e-20, 1.0, 1e18])
def test_zero_sources_list_every_key(hits, norm):
    """All their edges are 0: the zero keys' too, whose ties with the others the lowest key indices win."""
    assert all(hits(0.0, 0.0, 1, 0.0, norm))
    assert all(hits(-np.inf, 0.0, 1, 0.0, norm))
    assert not any(hits(0.5, 0.0, 1, 0.0, norm))


def test_zero_keys_are_listed_where_an_edge_of_0_reaches(hits):
    """A list of m entries holds the m largest edges only if none in it is below the bound."""
    bound = np.linspace(-1, 1, 16)
    assert hits(bound, 0.1, 1, 0.0, 0.0) == [int(b <= 0) for b in bound]
    assert all(hits(-np.inf, 0.1, 1, 0.0, 0.0))


def test_ordinary_keys_are_listed_where_the_edge_reaches(hits):
    """Against the edge in 64 bits: everything from the bound on, nothing further below than the slack and the
    rounding of a 32-bit multiply-add."""
    rng = np.random.default_rng(3)
    listed = 0
    for _ in range(2000):
        norm, inv = rng.uniform(1e-3, 30), rng.uniform(0.01, 30, 16).astype(np.float32)
        bound = rng.integers(-1024, 1025, 16) / 1024
        e = bound + rng.normal(0, 3e-5, 16)
        dot = (e * np.float32(norm) / inv).astype(np.float32)
        e = dot.astype(np.float64) * inv / float(np.float32(norm))
        got = np.array(hits(bound, inv, 1, dot, norm), dtype=bool)
        slack = 4e-6 + 1e-5 * np.abs(bound)
        assert got[e >= bound].all() and not got[e < bound - 2.1 * slack].any()
        listed += got.sum()
    assert 8000 < listed < 30000


@pytest.mark.parametrize("nan", [float(NAN[0]), float(NAN[1])])
def test_keys_with_nan_are_never_listed(hits, nan):
    assert not any(hits(np.linspace(-1, 1, 16), 0.1, 1, nan, nan))
    assert not any(hits(-np.inf, 0.1, 1, [0.0, nan] * 8, np.inf)[1::2])
