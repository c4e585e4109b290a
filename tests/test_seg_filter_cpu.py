"""The floating-point filter of the distance-to-segment test, compiled for the
host from the lines that the kernels use, against rational arithmetic: what it
decides is right, at the ends of segments much longer than the distance above
all.  Contraction into FMA changes which roundings happen, so it is compiled
without and with it.  Decisions are yes or no: no tolerance."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle.buffer import seg_within_exact

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_14362_amd", "csrc")
SOURCE = '#include "segfilter.h"\nextern "C" int seg_filter(double px, double py, double ax, double ay, double bx, ' \
         'double by, double r)\n{\n    return spade::seg_near_filter(px, py, spade::Seg{ax, ay, bx, by}, r * r);\n}\n'
FMA = open("/proc/cpuinfo").read().find(" fma ") >= 0


@pytest.fixture(scope="module", params=["plain", pytest.param("fma", marks=pytest.mark.skipif(not FMA, reason="no FMA"))])
def seg_filter(request, tmp_path_factory):
    d = tmp_path_factory.mktemp("segfilter")
    (d / "f.cpp").write_text(SOURCE)
    fp = ["-ffp-contract=off"] if request.param == "plain" else ["-mfma", "-ffp-contract=fast"]
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, "-shared",
                           "-fPIC"] + fp + ["-o", str(d / "f.so"), str(d / "f.cpp")])
    f = ctypes.CDLL(str(d / "f.so")).seg_filter
    f.argtypes, f.restype = [ctypes.c_double] * 7, ctypes.c_int
    return f


def _decided(f, cases):
    n = 0
    for c in cases:
        c = [float(v) for v in c]
        got = f(*c)
        assert got in (-1, 0, 1)
        if got >= 0:
            n += 1
            assert got == int(seg_within_exact(*c)), c
    return n


def test_known_ends(seg_filter):
    """p, a, b, r of points beside the far end of a long segment."""
    up = 1.0 + 1e-11
    _decided(seg_filter, [
        (-9e-10, 5e-5, -1e7, 0, 0, 0, 5e-5 * up), (-9e-7, 0.1, -1e10, 0, 0, 0, 0.1 * up),
        (2.395740662435006e-11, -9.081319519216338e-08, -626933.8878006589, -1.3669754518551256, 0, 0,
         9.081319535221679e-08),
        (500000.66551455046, 500000.0072300682, -241033.17544444726, 499993.5385700445, 500000.66551455046,
         500000.00723007496, 6.752088665941962e-09)])


@pytest.mark.parametrize("shift", [0.0, 5e5])
def test_ends_of_long_segments(seg_filter, shift):
    """Points within 20 r of an end, a step along the segment that is of the
    order of the rounding of its length, and the distance chosen between the
    end's and the line's."""
    rng = np.random.default_rng(17)
    cases = []
    for _ in range(6000):
        length, r = 10.0 ** rng.uniform(0, 7), 10.0 ** rng.uniform(-9, 1)
        th = rng.uniform(0, 2 * np.pi) if rng.random() < 0.6 else rng.integers(0, 4) * np.pi / 2
        co, si = np.cos(th), np.sin(th)
        e = np.array([co, si]) * length
        b = rng.uniform(-1, 1, 2) * shift
        along = rng.choice([-1, 1]) * length * 2.0 ** -53 * rng.uniform(0, 16)
        p = b + along * np.array([co, si]) + r * np.array([-si, co]) * rng.choice([1.0, rng.uniform(0, 20)])
        end = p - b
        near = abs(end[0] * -si + end[1] * co)      # from the line
        pick = rng.choice([near, np.hypot(*end), (near + np.hypot(*end)) / 2])
        pick *= 1.0 + rng.choice([-1, 1]) * 10.0 ** rng.uniform(-15, -9)
        cases.append((*p, *(b - e), *b, pick) if rng.random() < 0.7 else (*p, *b, *(b - e), pick))
    _decided(seg_filter, cases)


def test_ordinary_segments(seg_filter):
    """Segments, distances and points of like size: nearly all are decided."""
    rng = np.random.default_rng(18)
    v = rng.uniform(-100, 100, (3000, 6))
    r = rng.uniform(0, 60, 3000)
    assert _decided(seg_filter, [(*a, b) for a, b in zip(v, r)]) > 2990


@pytest.mark.parametrize("scale", [1e-180, 1e-130, 1e120, 1e160])
def test_ranges(seg_filter, scale):
    """Products that leave the normal range are left to the exact test."""
    rng = np.random.default_rng(19)
    v = rng.uniform(-1, 1, (400, 7))
    _decided(seg_filter, [(*(c[:6] * scale), abs(c[6]) * scale) for c in v])
    _decided(seg_filter, [(c[0], c[1], *(c[2:6] * scale), abs(c[6])) for c in v])
