"""No kernel of libblink.so asks for private memory (registers spilled to it, or
arrays indexed at run time). The runtime provides private memory by allocating it
on the device when such a kernel first runs on a queue, and the library promises
calls that allocate nothing. Read from the built library's own kernel metadata."""
import os
import re
import subprocess

import pytest

from paper_2405_13478_amd import build

LLVM = "/opt/rocm/llvm/bin"


def _kernels(tmp):
    tool = lambda name, *args: subprocess.run([os.path.join(LLVM, name), *args], check=True, capture_output=True,  # noqa: E731
                                              text=True).stdout
    fat, obj = os.path.join(tmp, "fat"), os.path.join(tmp, "gfx950.o")
    tool("llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, build.LIB, os.path.join(tmp, "copy.so"))
    tool("clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat, "--output=" + obj,
         "--targets=hipv4-amdgcn-amd-amdhsa--gfx950")
    notes = tool("llvm-readelf", "--notes", obj)
    # keys of a kernel's entry come in alphabetical order: its name before its private segment
    return re.findall(r"\.name: +(\S+)\n(?:(?!\.name:).)*?\.private_segment_fixed_size: +(\d+)", notes, re.S)


def test_no_kernel_uses_private_memory(tmp_path):
    if not os.path.exists(build.LIB) or not os.path.exists(os.path.join(LLVM, "clang-offload-bundler")):
        pytest.skip("needs the built library and ROCm's object tools")
    kernels = _kernels(str(tmp_path))
    assert len(kernels) > 100
    assert [k for k in kernels if int(k[1]) > 0] == []
