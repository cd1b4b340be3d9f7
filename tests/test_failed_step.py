"""A HIP call that fails in the middle of a step (csrc/mlda.hip): the state that is installed next is the state that was handed
over.  The library's host code is linked with a stand-in for the HIP runtime, whose launches do nothing, whose copies are
done at once, and of which the n-th launch can be told to fail."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1803_04631_amd._build import CSRC

STAND_IN = r'''
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
struct Launch { char name[64]; int failed; long long value; };
static struct Launch launches[4096];
static int n_launches = 0;
static const void* kernels[1024];
static const char* names[1024];
static int n_kernels = 0;
static int left = -1;                   // launches before the one that fails; negative: none does
static hipError_t last = hipSuccess;
static char somewhere[256];
extern "C" {
char FATBIN[16];
void fail_after(int launches) { left = launches; }
int launches_left() { return left; }
void forget_launches() { n_launches = 0; }
int launched(int i, char* name, int* failed, long long* value) {
    if (i >= n_launches) return 0;
    strcpy(name, launches[i].name); *failed = launches[i].failed; *value = launches[i].value;
    return 1;
}
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void** args, size_t, hipStream_t) {
    const int fails = left >= 0 && left-- == 0;
    struct Launch* l = &launches[n_launches < 4095 ? n_launches++ : 4095];
    l->name[0] = 0; l->failed = fails; l->value = 0;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i] == kernel) strncpy(l->name, names[i], 63);
    // whether the totals are cleared by it; PhiArgs::n_changed
    if (strstr(l->name, "zero_sums_kernel")) l->value = *(void**)args[3] != 0;
    if (strstr(l->name, "phi_tile_kernel")) l->value = ((int*)args[0])[4];
    if (fails) return last = hipErrorLaunchFailure;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* p; return &p; }
void __hipRegisterFunction(void**, const void* host, char* name, const char*, unsigned, void*, void*, void*, void*, int*) {
    kernels[n_kernels] = host; names[n_kernels++] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 100000;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = somewhere; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)somewhere; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)somewhere; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n ? n : 1, 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (n_launches < 4095) {
        struct Launch* l = &launches[n_launches++];
        strcpy(l->name, kind == hipMemcpyDeviceToHost ? "copy down" : "copy up"); l->failed = 0; l->value = (long long)n;
    }
    memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyWithStream(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memmove(d, s, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) { memset(a, 0, sizeof *a); a->type = hipMemoryTypeDevice; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)somewhere; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-c",
                           os.path.join(CSRC, "mlda.hip"), "-o", str(d / "mlda.o")])
    names = subprocess.check_output(["nm", "-u", str(d / "mlda.o")], text=True).split()
    fatbin = [n for n in names if n.startswith("__hip_fatbin")]
    (d / "hip.cpp").write_text(STAND_IN.replace("FATBIN", fatbin[0] if fatbin else "no_fatbin"))
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", str(d / "hip.cpp"),
                           str(d / "mlda.o"), "-lpthread", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", str(d / "mlda.so")])
    return ctypes.CDLL(str(d / "mlda.so"))


def launches_of(lib):
    """(kernel, whether its launch failed, value) of the launches since forget_launches."""
    name, failed, value = ctypes.create_string_buffer(64), ctypes.c_int(), ctypes.c_longlong()
    found = []
    while lib.launched(len(found), name, ctypes.byref(failed), ctypes.byref(value)):
        found.append((name.value.decode(), bool(failed.value), value.value))
    return found


class Model:
    def __init__(self, lib, doc_ptr, words, V, K, chunks):
        self.lib, self.doc_ptr, self.words = lib, doc_ptr, words
        self.ctx = ctypes.c_void_p()
        n = ctypes.c_size_t()
        D, seed = ctypes.c_int64(len(doc_ptr) - 1), ctypes.c_uint64(1)
        a, b = ctypes.c_double(0.5), ctypes.c_double(0.01)
        dp, wp = ctypes.c_void_p(doc_ptr.ctypes.data), ctypes.c_void_p(words.ctypes.data)
        if chunks > 1:
            assert lib.mlda_workspace_bytes_streamed(dp, D, V, K, chunks, ctypes.byref(n)) == 0
        else:
            assert lib.mlda_workspace_bytes(D, ctypes.c_int64(len(words)), V, K, ctypes.byref(n)) == 0
        self.memory = np.zeros(n.value + 256, dtype=np.uint8)
        at = ctypes.c_void_p((self.memory.ctypes.data + 255) // 256 * 256)
        if chunks > 1:
            rc = lib.mlda_create_streamed(ctypes.byref(self.ctx), dp, wp, D, V, K, a, b, seed, chunks, at, n, None)
        else:
            rc = lib.mlda_create(ctypes.byref(self.ctx), dp, wp, D, V, K, a, b, seed, at, n, None)
        assert rc == 0
        assert lib.mlda_init_random(self.ctx) == 0

    def close(self):
        self.lib.mlda_destroy(self.ctx)


@pytest.mark.parametrize("chunks", [2, 3, 5, 8])
@pytest.mark.parametrize("loglik", [0, 1])
def test_assignments_installed_after_a_failed_step(lib, chunks, loglik):
    rng = np.random.default_rng(chunks)
    V, K = 40, 12
    doc_ptr = np.concatenate([[0], np.cumsum(rng.integers(1, 30, 60))]).astype(np.int64)
    words = rng.integers(V, size=doc_ptr[-1]).astype(np.int32)
    z = rng.integers(1, K, size=doc_ptr[-1]).astype(np.uint16)
    failed = 0
    for launches in range(1000):
        m = Model(lib, doc_ptr, words, V, K, chunks)
        lib.fail_after(launches)
        rc = lib.mlda_step(m.ctx, 2, loglik)
        reached = lib.launches_left() < 0
        lib.fail_after(-1)
        lib.hipGetLastError()
        assert lib.mlda_set_assignments(m.ctx, ctypes.c_void_p(z.ctypes.data), 0) == 0
        got = np.zeros_like(z)
        assert lib.mlda_get_assignments(m.ctx, ctypes.c_void_p(got.ctypes.data)) == 0
        m.close()
        assert np.array_equal(got, z), (launches, rc)
        failed += rc != 0
        if not reached:
            break
    assert failed > 5 * chunks and rc == 0


def corpus(seed, V, T_most=30):
    rng = np.random.default_rng(seed)
    doc_ptr = np.concatenate([[0], np.cumsum(rng.integers(1, T_most, 60))]).astype(np.int64)
    return doc_ptr, rng.integers(V, size=doc_ptr[-1]).astype(np.int32)


@pytest.mark.parametrize("chunks,tokens", [(2, 5000), (3, 400000), (6, 900000), (7, 5000)])
def test_when_new_assignments_start_down(lib, chunks, tokens):
    """Behind the uploads of the next chunk (in a hardware queue that they share, the uploads would otherwise wait for the chunk's
    kernels), and before the next chunk's kernels (the upload after the next waits for the copy)."""
    V, K = 40, 12
    doc_ptr = np.arange(0, chunks * tokens + 1, 100, dtype=np.int64)
    words = np.random.default_rng(0).integers(V, size=doc_ptr[-1]).astype(np.int32)
    m = Model(lib, doc_ptr, words, V, K, chunks)
    lib.forget_launches()
    assert lib.mlda_step(m.ctx, 2, 0) == 0
    found = [(name, value) for name, _, value in launches_of(lib)]
    m.close()
    down = [i for i, (name, _) in enumerate(found) if name == "copy down"]
    assert [found[i][1] for i in down] == [2 * tokens] * (2 * chunks)
    assert down[-1] == len(found) - 1                               # (no chunk follows)
    for i in down[:-1]:
        assert found[i - 1] == ("copy up", 2 * tokens) and found[i - 2][0] == "copy up"
        made = max(j for j in range(i) if "to_doc_major" in found[j][0])
        assert not any("sample" in name or "theta" in name or "pair" in name for name, _ in found[made:i])
        assert "copy" not in found[i + 1][0]


def test_totals_are_cleared_after_a_failed_step(lib):
    """The topic totals are added to.  Where one launch rebuilds phi and theta it also clears the totals that nobody reads any more;
    if it fails they are as they were, and the next rebuild has to clear those that it adds to."""
    V, K = 40, 12
    doc_ptr, words = corpus(7, V)
    z = (np.arange(doc_ptr[-1]) % K).astype(np.uint16)
    failed_rebuilds = 0
    for launches in range(1000):
        lib.forget_launches()
        m = Model(lib, doc_ptr, words, V, K, 1)
        lib.fail_after(launches)
        rc = lib.mlda_step(m.ctx, 3, 1)
        reached = lib.launches_left() < 0
        lib.fail_after(-1)
        lib.hipGetLastError()
        cleared = False
        for name, failed, _ in launches_of(lib):
            if "phi_tile" in name:                  # takes what is cleared into use
                cleared = False
            elif "theta" in name or "rebuild_kernel" in name:
                cleared = not failed
                failed_rebuilds += failed
        lib.forget_launches()
        assert lib.mlda_set_assignments(m.ctx, ctypes.c_void_p(z.ctypes.data), 0) == 0
        clears = [value for name, _, value in launches_of(lib) if "zero_sums" in name]
        m.close()
        assert clears == ([] if cleared else [1]), (launches, rc)
        if not reached:
            break
    assert failed_rebuilds == 3 and rc == 0


@pytest.mark.parametrize("installed", [False, True])
def test_rows_of_phi_are_written_anew_after_a_failed_call(lib, installed):
    """Beyond 4,096 topics a step changes the cells of a word's old and new topics and leaves the rest of its row.  A rebuild
    that has not gone through, a step's or that of an installed state, leaves rows of other assignments: the next one writes
    them whole."""
    V, K = 40, 5000
    doc_ptr, words = corpus(7, V)
    z = (np.arange(doc_ptr[-1]) % K).astype(np.uint16)
    n_words = len(np.unique(words))
    assert np.bincount(words).max() <= K // 64
    anew = 0
    for launches in range(1000):
        lib.forget_launches()
        m = Model(lib, doc_ptr, words, V, K, 1)
        lib.fail_after(launches)
        if installed:
            rc = lib.mlda_set_assignments(m.ctx, ctypes.c_void_p(z.ctypes.data), 0)
        else:
            rc = lib.mlda_step(m.ctx, 3, 1)
        reached = lib.launches_left() < 0
        lib.fail_after(-1)
        lib.hipGetLastError()
        whole = True            # a rebuild of phi has been followed by one of theta
        for name, failed, _ in launches_of(lib):
            if "phi_tile" in name:
                whole = False
            elif "theta_r" in name and not failed:
                whole = True
        lib.forget_launches()
        assert lib.mlda_step(m.ctx, 2, 0) == 0
        changed = [value for name, _, value in launches_of(lib) if "phi_tile" in name]
        m.close()
        assert changed == ([n_words, n_words] if whole and not (installed and rc) else [0, n_words]), (launches, rc)
        anew += changed[0] == 0
        if not reached:
            break
    assert anew >= (2 if installed else 6) and rc == 0
