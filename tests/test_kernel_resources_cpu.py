"""What the compiler made of the kernels, read from the metadata of the built
library's own code object: properties that speed or safety rest on and that an
innocent edit can lose."""
import os
import struct
import subprocess

import pytest
import yaml

from paper_1905_12948_amd import build

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
EM_AMDGPU = 224


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> metadata of every kernel in libgmc.so."""
    if not os.path.exists(READELF) or not os.path.exists(build.LIB):
        pytest.skip("needs llvm-readelf and a built library")
    with open(build.LIB, "rb") as f:
        blob = f.read()
    out, at = {}, 0
    tmp = tmp_path_factory.mktemp("code")
    while True:
        at = blob.find(b"\x7fELF", at + 1)  # the library itself starts at 0
        if at < 0:
            return out
        if struct.unpack_from("<H", blob, at + 18)[0] != EM_AMDGPU:
            continue
        path = str(tmp / ("%d.elf" % at))
        with open(path, "wb") as f:
            f.write(blob[at:])
        text = subprocess.run([READELF, "--notes", path], check=True, capture_output=True, text=True).stdout
        for doc in text.split("---\n")[1:]:
            for k in yaml.safe_load(doc.split("\n...")[0])["amdhsa.kernels"]:
                out[k[".name"]] = k


def named(kernels, part):
    got = [k for n, k in kernels.items() if part in n]
    assert got, "no kernel named like " + part
    return got


def test_dynamic_lds_of_the_one_workgroup_selection_is_16_byte_aligned(kernels):
    # its dynamic array follows the static ones and is cleared with 16-byte stores
    for k in named(kernels, "topk_solo_kernel"):
        assert k[".group_segment_fixed_size"] % 16 == 0, (k[".name"], k[".group_segment_fixed_size"])


def test_the_copy_keeps_seven_wavefronts_per_simd(kernels):
    # 512 registers per lane and SIMD, allocated by eights; no scratch
    for k in named(kernels, "topk_copy_pass1_kernelILb0ELb0E"):
        assert k[".vgpr_count"] <= 72 and k[".private_segment_fixed_size"] == 0, k[".vgpr_count"]
        assert 7 * k[".group_segment_fixed_size"] <= 160 * 1024
