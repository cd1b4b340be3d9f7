"""LDS of the ranked theta rebuild (csrc/kernels_rebuild.hpp), on the host: where several waves share a workgroup, each wave's
part begins behind the others', and its mark words and cells are read and written 16 bytes at a time."""
import ctypes
import os
import subprocess

import pytest

from paper_1803_04631_amd._build import CSRC, HIPCC_FLAGS

SOURCE = '''#include <hip/hip_runtime.h>
#include "kernels_rebuild.hpp"
using namespace mlda;
// the first place in LDS (byte offset) of those that are accessed by 16 bytes and are not at a multiple of 16, or -1
extern "C" long long misaligned(int32_t K, long long longest, int docs) {
    const size_t wave_bytes = theta_rank_wave_bytes(K, longest, docs);
    for (int wave = 0; wave < 4; ++wave)
        for (int part = 0; part < docs; ++part) {
            const size_t words = kThetaLgTable * 8 + wave * wave_bytes + (size_t)part * theta_rank_words(K) * 8;
            const size_t cells = kThetaLgTable * 8 + wave * wave_bytes + (size_t)docs * theta_rank_words(K) * 8 +
                                 (size_t)part * theta_rank_cells(K, longest, docs) * 4;
            if (words % 16) return (long long)words;
            if (cells % 16) return (long long)cells;
        }
    return -1;
}
extern "C" long long spare(int32_t K, long long longest, int docs, int waves) {     // bytes of a launch behind the last wave's part
    return (long long)theta_rank_lds_bytes(K, longest, docs, waves) -
           (long long)(kThetaLgTable * 8 + (size_t)waves * theta_rank_wave_bytes(K, longest, docs)) ;
}
extern "C" long long unused(int32_t K, long long longest, int docs) {               // bytes of a wave's part behind its stage
    return (long long)theta_rank_wave_bytes(K, longest, docs) -
           docs * (theta_rank_words(K) * 8LL + theta_rank_cells(K, longest, docs) * 4LL + theta_rank_stage(longest, docs) * 2LL);
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("theta_rank")
    (d / "t.hip").write_text(SOURCE)
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *HIPCC_FLAGS, "-I" + CSRC, "-o", str(d / "t.so"), str(d / "t.hip")])
    lib = ctypes.CDLL(str(d / "t.so"))
    for f, n in ((lib.misaligned, 3), (lib.spare, 4), (lib.unused, 3)):
        f.restype = ctypes.c_longlong
        f.argtypes = [ctypes.c_int32, ctypes.c_longlong, ctypes.c_int, ctypes.c_int][:n]
    return lib


@pytest.mark.parametrize("docs", [1, 2])
def test_every_wave_begins_at_a_multiple_of_16(lib, docs):
    for K in (1, 3, 31, 33, 453, 999, 1024, 1025, 1500, 2047, 3072, 40000, 65535):
        for longest in [*range(0, 700), *range(2040, 2060), 2175, 2176, 2180, 3071, 3072]:
            assert lib.misaligned(K, longest, docs) == -1, (K, longest)
            assert lib.spare(K, longest, docs, 1) == lib.spare(K, longest, docs, 4) == 0
            assert 0 <= lib.unused(K, longest, docs) < 16
