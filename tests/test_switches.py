"""The environment switches' values (csrc/switches.hpp), compiled for the host: what is not a number in its range counts as none."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = '''#include "switches.hpp"
extern "C" int numbers(const char* t, int n, int64_t lo, int64_t hi, int64_t* v) { return mlda::switch_numbers(t, n, lo, hi, v); }
'''


@pytest.fixture(scope="module")
def numbers(tmp_path_factory):
    d = tmp_path_factory.mktemp("switches")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_1803_04631_amd", "csrc"),
                           "-o", str(d / "s.so"), str(d / "s.cpp")])
    f = ctypes.CDLL(str(d / "s.so")).numbers
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_char_p, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]

    def call(text, n, lo, hi):
        v = (ctypes.c_int64 * 4)(-7, -7, -7, -7)
        ok = f(None if text is None else text.encode(), n, lo, hi, ctypes.addressof(v))
        return tuple(v[:n]) if ok else (None if list(v) == [-7] * 4 else "stored")
    return call


def test_numbers_in_their_range(numbers):
    assert numbers("0", 1, 0, 2**63 - 1) == (0,)
    assert numbers("200000000", 1, 0, 2**63 - 1) == (200000000,)
    assert numbers("1024,64", 2, 0, 1024) == (1024, 64)


@pytest.mark.parametrize("text", [None, "", " ", "abc", "no", "12x", "1e8", "-1", "+5", " 5", "5 ", "0x10", "17",
                                  "99999999999999999999999"])
def test_everything_else_counts_as_none(numbers, text):
    assert numbers(text, 1, 0, 16) is None


@pytest.mark.parametrize("text", ["64", "64,", ",64", "64,64,64", "64;64", "64,x", "64, 64", "1025,1"])
def test_pairs(numbers, text):
    assert numbers(text, 2, 0, 1024) is None
