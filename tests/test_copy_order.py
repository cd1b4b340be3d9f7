"""copy_to_host_kernel (csrc/kernels_rebuild.hpp) tells the host by a flag that its bytes have arrived.  The flag is one thread's,
the bytes are all threads': on gfx950 a barrier does not wait for a wave's outstanding stores, so that every wave has to wait for
its own before it.  Shown in the code that the compiler makes of the kernel, here and without a GPU."""
import os
import re
import subprocess

import pytest

from paper_1803_04631_amd._build import CSRC, HIPCC_FLAGS


@pytest.fixture(scope="module")
def kernel(tmp_path_factory):
    d = tmp_path_factory.mktemp("copy")
    (d / "k.hip").write_text('#include <hip/hip_runtime.h>\n#include "kernels_rebuild.hpp"\n')
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-I" + CSRC, "--cuda-device-only", "-S",
                           "-o", str(d / "k.s"), str(d / "k.hip")])
    lines = (d / "k.s").read_text().splitlines()
    first = next(i for i, l in enumerate(lines) if re.match(r"_ZN4mlda19copy_to_host_kernel\w*:", l))
    last = next(i for i in range(first, len(lines)) if re.match(r"\s*s_endpgm", lines[i]))
    return [l.split(";")[0].strip() for l in lines[first:last + 1]]


def test_every_wave_waits_for_its_stores_before_the_barrier(kernel):
    barriers = [i for i, l in enumerate(kernel) if l.startswith("s_barrier")]
    stores = [i for i, l in enumerate(kernel) if re.match(r"(global|flat)_store_(byte|short|dword)", l)]
    waits = [i for i, l in enumerate(kernel) if l.startswith("s_waitcnt") and "vmcnt(0)" in l]
    assert len(barriers) == 1
    copies = [i for i in stores if i < barriers[0]]
    assert len(copies) >= 6         # four and one of 16 bytes, and the single bytes at the end
    # behind the last store, on the one way to the barrier: no branch target may lie between the wait and the barrier
    behind = [i for i in waits if copies[-1] < i < barriers[0]]
    assert behind, "\n".join(kernel[copies[-1]:barriers[0] + 1])
    assert not any(l.endswith(":") or l.startswith(("s_branch", "s_cbranch")) for l in kernel[behind[-1]:barriers[0]])
    # ... and the host's flag is the last store of all
    assert max(stores) > barriers[0] and [i for i in stores if i > barriers[0]][-1] == max(stores)
