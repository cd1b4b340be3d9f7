"""Where streamed chunks lie in their parts of the workspace (csrc/chunk_layout.hpp), compiled for the host.  A chunk's static
part is copied in while the assignments of the chunk before it in the same part may still be on their way out:
no chunk's buffers may reach any chunk's assignments, however different the chunks are."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = '''#include "chunk_layout.hpp"
#include <vector>
// per chunk: static part from .. to, whole layout to, assignments from .. to, all as offsets in a part; returns the part's size
extern "C" size_t lay_out(const int64_t* doc_ptr, int64_t D, int32_t M, const int64_t* words, int64_t slot_bytes, size_t* out) {
    std::vector<mlda::ChunkLayout> L;
    std::vector<int64_t> tokens;
    int64_t most_tokens = 0;
    size_t most_bytes = 0;
    for (int32_t m = 0; m < M; ++m) {
        const int64_t a = mlda::chunk_first(doc_ptr, D, M, m), b = mlda::chunk_first(doc_ptr, D, M, m + 1);
        tokens.push_back(doc_ptr[b] - doc_ptr[a]);
        L.push_back(mlda::chunk_layout(b - a, tokens[m], tokens[m] * 4 + (b - a) * slot_bytes, words[m], words[m], words[m], true));
        most_tokens = std::max(most_tokens, tokens[m]);
        most_bytes = std::max(most_bytes, L[m].total);
    }
    const mlda::StreamedSlot s = mlda::streamed_slot(most_tokens, most_bytes);
    for (int32_t m = 0; m < M; ++m, out += 5) {
        out[0] = s.chunk; out[1] = s.chunk + L[m].static_bytes; out[2] = s.chunk + L[m].total;
        out[3] = s.z_doc; out[4] = s.z_doc + tokens[m] * 2;
    }
    return s.total;
}
'''


@pytest.fixture(scope="module")
def lay_out(tmp_path_factory):
    d = tmp_path_factory.mktemp("chunk_layout")
    (d / "l.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_1803_04631_amd", "csrc"),
                           "-o", str(d / "l.so"), str(d / "l.cpp")])
    f = ctypes.CDLL(str(d / "l.so")).lay_out
    f.restype = ctypes.c_size_t
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]

    def call(lengths, chunks, words):
        doc_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
        words = np.asarray(words, dtype=np.int64)
        out = np.zeros((chunks, 5), dtype=np.uint64)
        total = f(doc_ptr.ctypes.data, len(lengths), chunks, words.ctypes.data, 32, out.ctypes.data)
        return out.astype(np.int64), total
    return call


def corpora():
    rng = np.random.default_rng(3)
    long_short = np.repeat([300, 3], [20000, 2000000])
    yield "long_then_short", long_short
    yield "short_then_long", long_short[::-1]
    yield "few_long_then_fives", np.repeat([300, 5], [2000, 120000])
    yield "then_empty", np.concatenate([np.full(3000, 200), np.zeros(400000, dtype=np.int64), np.full(3000, 200)])
    yield "few_documents", np.array([95817, 40000, 121924, 1, 44678, 0, 100000, 7])
    yield "alike", np.full(40000, 100)
    yield "ragged", rng.lognormal(4, 1.5, 5000).astype(np.int64)


@pytest.mark.parametrize("chunks", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("name,lengths", list(corpora()))
def test_no_chunk_reaches_the_assignments(lay_out, name, lengths, chunks):
    for words in (np.zeros(chunks), np.linspace(10, 200000, chunks), np.linspace(200000, 10, chunks)):
        out, total = lay_out(lengths, chunks, words)
        # (any chunk may follow any other: chunks without documents are left out, and an iteration starts over)
        static_from, _, layout_to, z_from, z_to = out.T
        assert z_from.min() >= 0 and layout_to.max() <= total and z_to.max() <= total
        assert z_to.max() <= static_from.min() or layout_to.max() <= z_from.min()
        assert np.all(static_from % 256 == 0) and np.all(z_from % 256 == 0)
