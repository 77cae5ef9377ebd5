"""What the compiler gave the kernels of the built library, read from its code objects' metadata: the
one-launch kernel keeps its transition columns in registers, and none of its forms may spill them."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2504_21411_amd", "libgsearch.so")
READELF = next((p for p in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf")) if p and os.path.exists(p)), None)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel symbol: {vgpr_count, vgpr_spill_count, private_segment_fixed_size}}"""
    if not READELF or not os.path.exists(LIB):
        pytest.skip("needs the built library and llvm-readelf")
    blob = open(LIB, "rb").read()
    d = tmp_path_factory.mktemp("code")
    out = {}
    starts = [m.start() for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", blob)]   # OS ABI 0x40: amdgpu_hsa
    for i, at in enumerate(starts):
        path = d / f"{i}.co"
        path.write_bytes(blob[at:])
        text = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for part in re.split(r"\n  - (?=\.)", text):
            sym = re.search(r"\.symbol:\s+(\S+)\.kd", part)
            if sym:
                out[sym.group(1)] = {k: int(re.search(rf"\.{k}:\s+(\d+)", part).group(1)) for k in
                                     ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    assert out, "no kernel metadata found"
    return out


def test_the_one_launch_kernel_keeps_nothing_in_scratch(kernels):
    small = {n: k for n, k in kernels.items() if "k_dp_small" in n}
    assert len(small) >= 16, sorted(kernels)
    for name, k in small.items():
        assert k["vgpr_count"] <= 128 and k["vgpr_spill_count"] == 0 and \
            k["private_segment_fixed_size"] == 0, (name, k)


def test_the_general_and_class_kernels_keep_nothing_in_scratch(kernels):
    """(one form of the bounded kernel does: two passes of eight targets with bounds per wave)"""
    for name, k in kernels.items():
        if re.search(r"k_dp_(push|tile|wide|class)", name):
            assert k["vgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0, (name, k)
