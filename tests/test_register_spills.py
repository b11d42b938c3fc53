"""Kernels whose registers are laid out to fit: a change (of the source or of the compiler) that makes one of them spill would
only be seen as a loss of time, or not at all.  The check reads the metadata of the library as it was built here."""
import os
import re
import subprocess

import pytest

import paper_2510_24061_amd as fq
from test_lds_waits import _code_objects

READELF = os.environ.get("LLVM_READELF", "/opt/rocm/llvm/bin/llvm-readelf")
# the initialization's kernels, the products, which hold operands of several steps, among them
INIT = ("apply_e_kernel", "apply_et_kernel", "apply_lower_kernel", "eigenvector_kernel", "factor_kernel", "gram_kernel",
        "init_residual_kernel", "jacobi_eig_kernel", "rotate_kernel", "settle_kernel", "sum_slices_kernel")


def _kernels(path, tmp_path):
    """mangled name -> (vector registers spilled, bytes of scratch)"""
    out = {}
    for i, obj in enumerate(_code_objects(path)):
        file = tmp_path / f"{i}.co"
        file.write_bytes(obj)
        text = subprocess.run([READELF, "--notes", str(file)], capture_output=True, text=True, check=True).stdout
        for entry in re.split(r"\n\s+- \.a", text)[1:]:
            fields = dict(re.findall(r"\.(name|vgpr_spill_count|private_segment_fixed_size):\s+(\S+)", entry))
            if len(fields) == 3:
                out[fields["name"]] = (int(fields["vgpr_spill_count"]), int(fields["private_segment_fixed_size"]))
    return out


def _spilling(kernels):
    return {n: k for n, k in kernels.items() if k != (0, 0) and any(re.search(rf"\d{base}(I|E)", n) for base in INIT)}


def test_the_check_itself():
    assert _spilling({"_ZN6falqon12_GLOBAL__N_114apply_e_kernelILi8EEEvPKf": (66, 220), "_ZN6falqon12_GLOBAL__N_115gemm_fp8_kernelILi2EE": (17, 72),
                      "_ZN6falqon12_GLOBAL__N_111gram_kernelEPKf": (0, 0)}) == {"_ZN6falqon12_GLOBAL__N_114apply_e_kernelILi8EEEvPKf": (66, 220)}


def test_the_kernels_of_the_initialization_spill_nothing(tmp_path):
    if not os.path.exists(fq.lib_path()):
        pytest.skip("library not built")
    kernels = _kernels(fq.lib_path(), tmp_path)
    for base, least in (("apply_e_kernel", 6), ("apply_et_kernel", 6), ("factor_kernel", 14), ("jacobi_eig_kernel", 14), ("gram_kernel", 2)):
        assert sum(bool(re.search(rf"\d{base}(I|E)", n)) for n in kernels) >= least, base
    bad = _spilling(kernels)
    assert not bad, bad
