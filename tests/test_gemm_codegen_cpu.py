"""What the compiler made of the main GEMM kernels, read from the object that the build leaves (its own gfx950 code): scalar
registers that are spilled are fetched back lane by lane, and where a group of kernel arguments is, in front of every store."""
import os
import re
import subprocess

import pytest

import paper_2412_19437_amd as pkg

OBJECT = os.path.join(os.path.dirname(pkg.__file__), "_build", "ds3_gemm.o")
LLVM = "/opt/rocm/llvm/bin"
LANE_READS = 600          # the kernels have 38 to 354; those whose epilogue reloaded the arguments had 661 to 1815


@pytest.mark.skipif(not os.path.exists(OBJECT) or not os.path.exists(f"{LLVM}/llvm-objdump"), reason="no object or no disassembler")
def test_epilogues_do_not_reload_the_kernel_arguments(tmp_path):
    fat, dev = tmp_path / "fat", tmp_path / "dev.o"
    run = lambda *a: subprocess.run([f"{LLVM}/{a[0]}", *map(str, a[1:])], check=True, capture_output=True, text=True).stdout
    run("llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", OBJECT, tmp_path / "copy.o")
    run("clang-offload-bundler", "--type=o", "--unbundle", f"--input={fat}", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
        f"--output={dev}")
    kernels = re.split(r"\n[0-9a-f]+ <(\S+)>:\n", run("llvm-objdump", "-d", "--no-show-raw-insn", dev))
    reads = {name: body.count("v_readlane_b32") for name, body in zip(kernels[1::2], kernels[2::2]) if "gemm_fp8_bs_kernel" in name}
    assert len(reads) >= 48
    assert {n: c for n, c in reads.items() if c > LANE_READS} == {}
