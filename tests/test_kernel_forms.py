"""Sizes that need little of a kernel have a kernel of their own: in one kernel with the rest, chosen at run time, they paid for
the registers, masks and code of all of it.  Registers are read from the built library's own metadata."""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


def _registers(tmp_path):
    from paper_2509_23472_amd import build
    if not os.path.exists(build.LIB_PATH):
        build.build_library(verbose=False)
    fat, obj = str(tmp_path / "fat"), str(tmp_path / "obj")
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, build.LIB_PATH, str(tmp_path / "copy")], check=True)
    subprocess.run([LLVM + "/clang-offload-bundler", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat,
                    "--output=" + obj, "--unbundle"], check=True)
    notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
    found = re.findall(r"\.name: +(\S+)\n.*?\.vgpr_count: +(\d+)\n +\.vgpr_spill_count: +(\d+)", notes, re.S)
    return {name: (int(count), int(spilled)) for name, count, spilled in found if ".kd" not in name}


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    if not os.path.exists(LLVM + "/clang-offload-bundler"):
        pytest.skip("no LLVM tools")
    return _registers(tmp_path_factory.mktemp("registers"))


@pytest.fixture(scope="module")
def vgprs(registers):
    return {name: count for name, (count, _) in registers.items()}


def test_float32_qr_of_few_columns(vgprs):
    for strips in (2, 4):                      # (eight strips fill the registers in either form)
        few = [v for n, v in vgprs.items() if "ortho_small_f64_kernelILi%dELb0" % strips in n]
        rows = [v for n, v in vgprs.items() if "ortho_small_f64_kernelILi%dELb1" % strips in n]
        assert len(few) == len(rows) == 1 and few[0] < rows[0], (strips, few, rows)
    few = [v for n, v in vgprs.items() if "chol_inverse_wave_kernelILi16ELb0" in n]
    rows = [v for n, v in vgprs.items() if "chol_inverse_wave_kernelILi16ELb1" in n]
    assert len(few) == len(rows) == 1 and few[0] < rows[0], (few, rows)


def test_factorisation_of_few_columns(vgprs):
    # (ortho_f64.h: 1, 4, 8, 12 and 16 blocks of 16 columns)
    of = {nbm: [v for n, v in vgprs.items() if "chol_reg_kernelILi%dE" % nbm in n] for nbm in (1, 4, 8, 12, 16)}
    assert all(len(v) == 1 for v in of.values()), of
    assert of[8][0] < of[12][0] < of[16][0], of


def test_spills_of_the_factorisation(registers):
    # nothing up to 192 columns; 17 blocks, with the first block row in LDS, not twice what 16 spill
    alone = {nbm: [v for n, v in registers.items() if "chol_reg_kernelILi%dE" % nbm in n] for nbm in (1, 4, 8, 12, 16, 17)}
    fused = {nj: [v for n, v in registers.items() if "chol_trsm_fused_kernelILi%dELi%dE" % ((nj + 3) // 4 * 4, nj) in n] for nj in range(1, 17)}
    assert all(len(v) == 1 for v in list(alone.values()) + list(fused.values())), (alone, fused)
    assert all(alone[nbm][0][1] == 0 for nbm in (1, 4, 8, 12)) and all(fused[nj][0][1] == 0 for nj in range(1, 13)), (alone, fused)
    assert 0 < alone[17][0][1] < 2 * alone[16][0][1] and alone[16][0][1] <= 32 and all(fused[nj][0][1] <= 32 for nj in range(13, 17)), (alone, fused)
