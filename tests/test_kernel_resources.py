"""Register use of compiled kernels, from the metadata of the objects the build leaves: no GPU."""
import os
import re
import shutil
import subprocess

import pytest

BUILD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2602_06071_amd", "_build")
LLVM = "/opt/rocm/llvm/bin"


def spills(obj, tmp_path):
    """{mangled kernel name: spilled vector registers} of a compiled translation unit."""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
    src = os.path.join(BUILD, obj)
    if not os.path.exists(src) or not all(shutil.which(t) for t in tools):
        pytest.skip("no build or no tools")
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([tools[0], f"--dump-section=.hip_fatbin={fat}", src, str(tmp_path / "copy.o")], check=True)
    subprocess.run([tools[1], "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}",
                    f"--output={code}"], check=True)
    notes = subprocess.run([tools[2], "--notes", code], check=True, capture_output=True, text=True).stdout
    out = {}
    for kernel in re.split(r"\n  - \.agpr_count", notes)[1:]:
        name = re.search(r"\.name:\s+(\S+)", kernel)
        out[name.group(1)] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    return out


@pytest.mark.parametrize("obj", ["k_ksplit_f16.o", "k_ksplit_bf16.o"])
def test_ksplit_kernels_of_unaligned_rows_spill_nothing_at_tiles_of_32_and_128_rows(obj, tmp_path):
    """(64 rows: two waves per SIMD leave too few registers at any ring depth.)"""
    unaligned = {k: v for k, v in spills(obj, tmp_path).items()
                 if re.search(r"ksplit_kernelI\w+Li[14]ELi4ELb[01]ELb1E", k)}
    assert len(unaligned) == 4 and set(unaligned.values()) == {0}, unaligned


def test_shared_phi_kernels_spill_only_for_unaligned_rows_of_64_and_128_row_tiles(tmp_path):
    """(There the alignment of the rows takes the registers that were left: 27 and 30 with 64 rows, 19 with 128.)"""
    found = {tuple(map(int, re.search(r"outs_kernelI\w+?Li(\d)ELi(\d)ELb([01])E", k).groups())) + (k,): v
             for k, v in spills("k_outs.o", tmp_path).items() if "outs_kernel" in k}
    assert len(found) == 24
    for (mt, _, unal, name), v in found.items():
        assert v <= (30 if unal and mt > 1 else 0), (name, v)


@pytest.mark.parametrize("obj", ["k_vector.o", "k_rows.o", "k_blockrow.o"])
def test_kernels_of_few_vectors_of_the_rows_layout_and_of_block_rows_spill_nothing(obj, tmp_path):
    """(Two registers in the rows kernel's output-stationary tiles of 128 rows and 128 examples, which fill the file.)"""
    found = spills(obj, tmp_path)
    assert found
    for name, v in found.items():
        assert v <= (2 if re.search(r"rows_kernelI\w+?Li4ELi4ELNS0_8RowsModeE1E", name) else 0), (name, v)


def test_dense_kernels_spill_nothing(tmp_path):
    """(Those of 512 columns fill 472 to 504 of a lane's 512 registers.)"""
    found = {k: v for k, v in spills("k_gauss.o", tmp_path).items() if "gauss_kernel" in k}
    assert len(found) == 20 and set(found.values()) == {0}, found
