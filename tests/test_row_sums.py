"""Sums over a theta row that hold no rounding (csrc/row_sums.hpp), on the CPU: the header's rule, compiled for the host,
against exact sums.  A token that shares the walk over its row gets the sums from it only where the rule
lets it, and they then have to be those of a walk of its own to the last bit, whatever the weights are."""
import ctypes
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCALE_LOG2 = -42        # what sums carry as a factor where weights are staged in fp64

SOURCE = '''#include "row_sums.hpp"
extern "C" uint32_t below(uint32_t least, int log2_scale) { return mlda::exact_sums_below(least, log2_scale); }
'''


@pytest.fixture(scope="module")
def below(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_sums")
    (d / "below.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "paper_1803_04631_amd", "csrc"),
                           "-o", str(d / "below.so"), str(d / "below.cpp")])
    f = ctypes.CDLL(str(d / "below.so")).below
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_uint32, ctypes.c_int]
    return f


def bits(w):
    return int(np.float32(w).view(np.uint32))


def upper_dword(x):
    return int(np.float64(x).view(np.uint64)) >> 32


def is_exact(below, row_sum, least, log2_scale):
    return upper_dword(np.ldexp(np.float64(row_sum), log2_scale)) < below(bits(least), log2_scale)


def walk(counts, weights, own, w_o):
    """A token's own walk: the own topic's other tokens with w_o, everything else with its weight (products are exact)."""
    acc, ends = np.float64(0), []
    for k, (c, w) in enumerate(zip(counts, weights)):
        acc = acc + np.float64(c - (k == own)) * np.float64(w_o if k == own else w)
        ends.append(acc)
    return ends


def shared_walk(counts, weights, own, w_o):
    """Every topic with its weight, in four lanes side by side; the own topic's share put right afterwards."""
    n = -(-len(counts) // 4)
    ends, before = [], np.float64(0)
    for lane in range(4):
        acc = np.float64(0)
        for k in range(lane * n, min(lane * n + n, len(counts))):
            acc = acc + np.float64(counts[k]) * np.float64(weights[k])
            ends.append(before + acc)
        before = before + acc
    row_sum = before
    c = np.float64(counts[own])
    shift = (c - 1) * np.float64(w_o) - c * np.float64(weights[own])
    return [e + (shift if k >= own else 0.0) for k, e in enumerate(ends)], row_sum


def rows(rng, decades, n_rows, largest_count):
    for _ in range(n_rows):
        n = int(rng.integers(2, 40))
        weights = (10.0 ** rng.uniform(-decades, 0, n)).astype(np.float32)
        counts = np.maximum(1, rng.geometric(1.0 / rng.uniform(1.01, largest_count), n))
        own = int(rng.integers(n))
        w_o = np.float32(weights[own] * rng.uniform(0.3, 1.0))
        yield counts, weights, own, w_o


# (weights over so many decades: at beta = 0.01 a word's lie within 6 to 8)
@pytest.mark.parametrize("log2_scale", [0, SCALE_LOG2])
@pytest.mark.parametrize("decades", [1, 4, 7, 8, 10, 30])
def test_shared_sums_are_those_of_a_walk_of_its_own(below, decades, log2_scale):
    rng = np.random.default_rng(decades)
    let = rounded = 0
    for counts, weights, own, w_o in rows(rng, decades, 1500, 40):
        ends = walk(counts, weights, own, w_o)
        shared, row_sum = shared_walk(counts, weights, own, w_o)
        if not is_exact(below, row_sum, min(weights.min(), w_o), log2_scale):
            rounded += shared != ends
            continue
        let += 1
        assert shared == ends
        true = sum(int(c) * Fraction(float(w)) for c, w in zip(counts, weights))
        assert Fraction(float(row_sum)) == true
    # the rule lets what real weights need, and where it does not, sums do round
    if decades <= 7:
        assert let > 1400
    if decades >= 10:
        assert rounded > 0


@pytest.mark.parametrize("least", [1.0, 0.75, 2.0 ** -20, 1e-8, float(np.float32(1.1754944e-38)), 1e-40, 0.0])
@pytest.mark.parametrize("log2_scale", [0, SCALE_LOG2])
def test_limit(below, least, log2_scale):
    """2^30 times the power of two below the least weight; 2^-96 for denormal weights and 0; never for what is no number."""
    w = np.float32(least)
    e = max(int(np.floor(np.log2(float(w)))) if w > 0 else -200, -126)
    limit = np.ldexp(1.0, e + 30)
    assert not is_exact(below, limit, w, log2_scale)
    assert is_exact(below, np.nextafter(limit, 0.0), w, log2_scale)
    assert is_exact(below, 0.0, w, log2_scale)
    assert not is_exact(below, np.inf, w, log2_scale) and not is_exact(below, np.nan, w, log2_scale)
