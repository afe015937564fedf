"""CPU-only checks of the compiled kernels: what a compute unit can hold of them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_00388_amd import binding as gk


def rocm_tool(name):
    hipcc = shutil.which("hipcc")
    at = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "llvm", "bin") if hipcc else None
    for path in (at, "/opt/rocm/llvm/bin"):
        if path and os.path.exists(os.path.join(path, name)):
            return os.path.join(path, name)
    pytest.skip(f"no {name}")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """What the compiler states of every kernel of the library, by name."""
    objdump, readelf = rocm_tool("llvm-objdump"), rocm_tool("llvm-readelf")
    if not os.path.exists(gk.LIB_PATH):
        from paper_2509_00388_amd import build
        build.build()
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(gk.LIB_PATH, where)
    subprocess.run([objdump, "--offloading", lib], cwd=where, check=True, capture_output=True)
    found, entry = {}, {}
    for name in sorted(os.listdir(where)):
        if not name.endswith("gfx950"):
            continue
        notes = subprocess.run([readelf, "--notes", name], cwd=where, check=True, capture_output=True, text=True).stdout
        for key, value in re.findall(r"^\s+(?:- )?\s*\.(\w+):\s+(\S+)$", notes, re.M):
            if key == "agpr_count":   # (the first of a kernel's entries)
                entry = {}
            entry[key] = value
            if key == "wavefront_size":
                found[entry["symbol"].removesuffix(".kd")] = entry
    assert found
    return found


@pytest.mark.parametrize("kernel,waves,variants", [("gemm_cosine_kernel", 2, 12), ("gemm_logits_kernel", 3, 12),
                                                   # (96 source rows in 250 of 256 registers, 16 triples a thread in all 128)
                                                   ("bound_filter_kernel", 2, 6), ("cosine_filter_kernel", 2, 4),
                                                   ("cosine_maxima_kernel", 2, 2), ("decay_radix_kernel", 4, 2)])
def test_kernels_hide_their_loads_behind_other_waves(kernels, kernel, waves, variants):
    """Every variant leaves a SIMD's 512 registers to so many waves, without spilling."""
    some = {name: k for name, k in kernels.items() if kernel in name}
    assert len(some) >= variants
    for name, k in some.items():
        assert int(k["vgpr_count"]) <= 512 // waves // 8 * 8, (name, k["vgpr_count"])
        assert int(k["vgpr_spill_count"]) == 0 and int(k["private_segment_fixed_size"]) == 0, name
