"""Properties of the device primitives that the compiled code shows without a GPU."""

import os
import re
import subprocess

import pytest

from paper_2606_03075_amd import build

SOURCE = """
#include "tgvkv_device.h"
__global__ void mark_and_look(unsigned long long* marks, int mine, int other, unsigned long long call, int* seen) {
    __hip_atomic_store(marks + mine, call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tgvkv::wait_vmem_ordered();
    *seen = __hip_atomic_load(marks + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == call;
}
"""


def _hipcc():
    try:
        return build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")


def test_the_marks_of_split_decode_stay_in_order(tmp_path):
    """Store, wait, load: the compiler sees the wait as an access to all memory, so neither side may cross it; in the
    assembly the store is followed by the wait and that by the load."""
    src = tmp_path / "order.hip"
    src.write_text(SOURCE)
    flags = build.common_flags() + build.device_flags() + ["-x", "hip", "--cuda-device-only", "-S", str(src), "-o"]
    for more, parts in ((["-emit-llvm"], (r"store atomic i64", r'asm sideeffect "s_waitcnt vmcnt\(0\)", "[^"]*~\{memory\}',
                                         r"load atomic i64")),
                        ([], (r"global_store_dwordx2 .* sc1", r"s_waitcnt vmcnt\(0\)", r"global_load_dwordx2 .* sc1"))):
        out = tmp_path / "order.out"
        r = subprocess.run([_hipcc()] + flags + [str(out)] + more, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
        text = out.read_text()
        assert re.search(".*".join(parts), text, flags=re.S), text
        assert len(re.findall(parts[0], text)) == len(re.findall(parts[2], text)) == 1


def test_split_decode_waits_in_order():
    """The combination of split partials uses no other wait."""
    with open(os.path.join(build.CSRC, "decode.hip")) as f:
        text = f.read()
    assert text.count("wait_vmem_ordered();") == 2 and "wait_vmem_all" not in text
