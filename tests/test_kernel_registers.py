"""What the compiler made of the library's kernels, from the metadata of the code object built here: none keeps registers in scratch
memory, and those whose launch rules count on a number of waves per SIMD can have them."""
import os
import re
import subprocess

import host_path

LLVM = "/opt/rocm/llvm/bin/"


def kernels(tmp_path):
    """{name with template arguments: {field: number}} of the kernels in the built library"""
    fat, obj = str(tmp_path / "fat"), str(tmp_path / "obj")
    subprocess.check_call(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", host_path.LIB, fat])
    subprocess.check_call([LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat, "--output=" + obj,
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
    notes = subprocess.check_output([LLVM + "llvm-readelf", "--notes", obj], text=True)
    out = {}
    for part in notes.split("- .agpr_count:")[1:]:
        name = subprocess.check_output(["c++filt", re.search(r"\.symbol:\s*(\S+)\.kd", part).group(1)], text=True)
        name = re.match(r"(?:void )?fs::(\w+(?:<[^(]*>)?)\(", name)
        if name:
            field = lambda f: int(re.search(rf"\.{f}:\s*(\d+)", part).group(1))
            out[name.group(1).replace(" ", "")] = {f: field(f) for f in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size",
                                                                         "group_segment_fixed_size")}
    return out


def test_registers(tmp_path):
    assert os.path.exists(host_path.LIB)
    ks = kernels(tmp_path)
    assert len(ks) > 40
    spilled = {n: k for n, k in ks.items() if k["vgpr_spill_count"] or k["private_segment_fixed_size"]}
    assert not spilled, spilled
    # 512 registers per lane of a SIMD: waves = 512 // registers, in eights
    waves = lambda n: 512 // (-(-ks[n]["vgpr_count"] // 8) * 8)
    for j in ("true", "false"):
        for f in ("true", "false"):
            n = f"k_solve_ws<{f},{j},3,true>"          # three blocks of four waves per CU of 160 KiB LDS
            assert waves(n) >= 3 and 3 * ks[n]["group_segment_fixed_size"] <= 160 << 10, (n, ks[n])
    for n in ("k_grad_records<true,1,1>", "k_grad_records<false,1,1>"):
        assert waves(n) >= 4, (n, ks[n])
