"""What the compiler made of the kernels, from the metadata of the library that this tree builds."""
import os
import re
import subprocess

import pytest

import paper_2104_10716_amd as es
from paper_2104_10716_amd import build

LLVM = "/opt/rocm/llvm/bin"


def _kernels(tmp_path):
    """{kernel: (bytes of scratch memory, vector registers spilled)}"""
    es.load_library()
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={bundle}", build.LIB, os.devnull], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    f"--input={bundle}", f"--output={code}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    found = re.findall(r"\.name: +(_Z\w+kernel\w+)\n.*?\.private_segment_fixed_size: +(\d+)\n.*?\.vgpr_spill_count: +(\d+)\n",
                       notes, re.S)
    return {name: (int(scratch), int(spilled)) for name, scratch, spilled in found}


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/clang-offload-bundler"), reason="no LLVM tools")
def test_no_kernel_spills(tmp_path):
    """A spill in these kernels' gather loops costs more than the waves it was bought for."""
    kernels = _kernels(tmp_path)
    assert len(kernels) > 200 and any("es_pull_kernel" in k for k in kernels)
    assert {k: v for k, v in kernels.items() if v != (0, 0)} == {}
