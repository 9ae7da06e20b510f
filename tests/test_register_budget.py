"""The 256x256 bf16 product kernels must leave room for the weight-update kernel on the same compute unit.

Two wavefronts of a product workgroup share a SIMD's 512 registers per lane with the update kernel's wavefronts, which
need 64: above 224 registers per lane (or with spills) the update no longer runs beside the products and a training step
of the large configurations gets ~10 % slower without any test of the arithmetic noticing.  The kernel of small layers holds
all its tile variants, and its epilogue's operands over the k-loop: a spill there would cost every launch.  This compiles the
device code with the library's own flags and reads the register counts out of the code objects' metadata.  What the
kernels' assembly writes beside its operands has to be known to the compiler; that is read out of the intermediate code.
"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2403_11204_amd import build

def metadata_of(unit):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "unit.s")
        cmd = [build.hipcc()] + [a for a in build.COMMON if a != "-fPIC"] + build.UNITS[unit] + ["--cuda-device-only", "-S", os.path.join(build.CSRC, unit), "-o", out]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout[-2000:]
        text = open(out).read()
    meta = text[text.index("amdhsa.kernels"):]
    kernels = {}
    for entry in meta.split("- .agpr_count")[1:]:
        name = re.search(r"\.name:\s+(\S+)", entry).group(1)
        kernels[name] = {k: int(re.search(r"\.%s:\s+(\d+)" % k, entry).group(1))
                         for k in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    return kernels


@pytest.fixture(scope="module")
def kernel_metadata():
    return metadata_of("gemm.hip")


def test_big_product_kernels_fit_beside_the_update_kernel(kernel_metadata):
    big = {n: v for n, v in kernel_metadata.items() if "gemm_nt_big_kernel" in n}
    assert len(big) == 4, sorted(big)          # forward, data gradient, weight gradient, weight gradient + update
    for name, v in big.items():
        assert v["vgpr_count"] <= 224, (name, v)
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)


def test_long_product_kernels_fit_beside_the_update_kernel(kernel_metadata):
    long = {n: v for n, v in kernel_metadata.items() if "gemm_nt_long_kernel" in n}
    assert len(long) == 3, sorted(long)        # forward, data gradient, weight gradient
    for name, v in long.items():
        assert v["vgpr_count"] <= 448, (name, v)           # one wavefront of a workgroup on a SIMD, and one of the update's
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)


def test_no_product_kernel_spills(kernel_metadata):
    for name, v in kernel_metadata.items():
        if "gemm_nt" in name:
            assert v["vgpr_spill_count"] == 0, (name, v)


def test_the_kernels_of_small_layers_do_not_spill():
    small = metadata_of("gemm_small.hip")
    assert sum("small_group_kernel" in n for n in small) == 2 and sum("small_product_kernel" in n for n in small) == 12, sorted(small)
    for name, v in small.items():
        assert v["vgpr_count"] <= 128, (name, v)           # 4 workgroups of 4 wavefronts per compute unit
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)


def test_the_kernels_of_product_pairs_fit_their_workgroups():
    pair = metadata_of("gemm_pair.hip")
    assert len(pair) == 8, sorted(pair)
    for name, v in pair.items():
        assert v["vgpr_count"] <= (168 if "Li64E" in name else 256), (name, v)      # 3 and 2 workgroups of 4 wavefronts per compute unit
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)


def test_the_update_kernel_fits_beside_the_products():
    update = {n: v for n, v in metadata_of("elementwise.hip").items() if "sgd_update_strided_kernel" in n}
    assert len(update) == 2, sorted(update)
    for name, v in update.items():
        assert v["vgpr_count"] <= 64, (name, v)
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)


@pytest.mark.parametrize("unit", sorted(build.UNITS))
def test_assembly_names_what_it_writes(unit):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "unit.ll")
        cmd = [build.hipcc()] + [a for a in build.COMMON if a != "-fPIC"] + build.UNITS[unit] + ["--cuda-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", os.path.join(build.CSRC, unit), "-o", out]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout[-2000:]
        statements = re.findall(r'asm (?:sideeffect )?"([^"]*)", "([^"]*)"', open(out).read())
    assert len(statements) > 0 or unit != "gemm.hip"
    for text, constraints in statements:
        for line in re.split(r"\\0A(?:\\09)?", text):
            op, _, operands = line.strip().partition(" ")
            written = operands.split(",")[0].strip()
            if re.fullmatch(r"m0|vcc|exec|[sva]\d+", written):
                assert "~{%s}" % written in constraints, (line, constraints)
            if re.match(r"s_(add|sub|and|or|xor|lsh[lr]|cmp)", op):
                assert "~{scc}" in constraints, (line, constraints)
