"""Registers of the reverse collide kernel as compiled for gfx950: no storage and neither offset width may
spill to scratch memory. The FP64 kernel needs more registers than three waves per SIMD leave it, with
64-bit offsets as with 32-bit ones. CPU only (a compilation of the kernel alone, nothing runs)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """#include <hip/hip_runtime.h>
#include "adjoint_kernels.hpp"
%s
"""


def test_reverse_collide_does_not_spill(tmp_path):
    from paper_2608_15781_amd import build

    modes = {0: "double", 1: "float", 2: "float", 3: "float", 4: "double", 5: "float", 6: "float", 7: "float"}
    src = tmp_path / "kernels.hip"
    src.write_text(SOURCE % "\n".join("template __global__ void lbm::k_adj_collide<%d>(lbm::StepArgs<%d>, lbm::AdjArgs<%s>);"
                                      % (m, m, t) for m, t in modes.items()))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([build.hipcc()] + flags + ["-I" + os.path.join(ROOT, "paper_2608_15781_amd", "csrc"),
                                                  "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
                                                  "-o", str(tmp_path / "kernels.o"), str(src)],
                       capture_output=True, text=True, check=True)
    scratch, name = {}, None
    for line in r.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line):
            scratch[name] = int(m.group(1))
    found = {int(m.group(1)): v for k, v in scratch.items() if (m := re.search(r"k_adj_collideILi(\d)E", k))}
    assert found == {m: 0 for m in modes}, found
