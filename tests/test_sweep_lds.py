"""The static LDS that the sweep's histogram plan leaves room for is what the compiled kernels hold."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_26799_amd", "csrc")
OBJ = os.path.join(ROOT, "paper_2604_26799_amd", "_build", "sweep.hip.o")
LLVM = "/opt/rocm/llvm/bin"

DRIVER = """
#include <cstdio>
#include <cstdlib>
#include "sweep.h"
int main(int argc, char** argv) {
    for (int i = 1; i + 1 < argc; i += 2)
        std::printf("%d\\n", mgs::static_lds_bytes(std::atoi(argv[i]), std::atoi(argv[i + 1])));
}
"""


@pytest.mark.skipif(not (os.path.exists(OBJ) and os.path.exists(os.path.join(LLVM, "llvm-readelf"))),
                    reason="needs the built object and the LLVM tools")
def test_static_lds_of_every_kernel(tmp_path):
    fat, co, exe = (str(tmp_path / n) for n in ("fat", "co", "driver"))
    run = lambda *cmd: subprocess.run(cmd, check=True, capture_output=True, text=True).stdout
    run(f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", OBJ, str(tmp_path / "copy.o"))
    run(f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={co}",
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950")
    notes = run(f"{LLVM}/llvm-readelf", "--notes", co)
    held = {}
    for part in notes.split(".group_segment_fixed_size:")[1:]:
        m = re.search(r"\.name:\s+_ZN3mgs12sweep_kernelILi(\d+)ELi(\d+)ELb([01])ELi(\d+)E", part)
        if m:
            held[tuple(int(v) for v in m.groups())] = int(part.split()[0])
    assert len(held) >= 20
    (tmp_path / "driver.cpp").write_text(DRIVER)
    run("/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-I", CSRC,
        str(tmp_path / "driver.cpp"), "-o", exe)
    kernels = sorted(held)
    planned = [int(v) for v in run(exe, *[str(v) for nt, _, _, sub in kernels for v in (nt, sub)]).split()]
    for kernel, plan in zip(kernels, planned):
        assert held[kernel] <= plan <= held[kernel] + 512, kernel
