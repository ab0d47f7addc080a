"""The step and reverse kernels read no unset value. A load masked off in some lanes leaves its destination
unset there, and a blend that drops it again is still undefined to the compiler, which may then drop
the blend, for an index as for a value. In the compiler's IR such a value is a phi with an undefined
operand; there may be none. CPU only (compiled to IR, nothing runs)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STEP = ["k_colour<%d, 256, false>", "k_colour<%d, 128, false>", "k_extrap<%d, false>", "k_normal<%d, false>",
        "k_collide<%d, false, true, 256, 0>", "k_collide<%d, false, false, 128, 0>"]
REVERSE = ["k_adj_collide<%d>", "k_adj_normal<%d>", "k_adj_colour<%d>", "k_adj_final<%d>", "k_adj_grad_ext<%d>"]


def test_no_phi_of_an_unset_value(tmp_path):
    from paper_2608_15781_amd import build

    lines = ["#include <hip/hip_runtime.h>", '#include "adjoint_kernels.hpp"']
    for mode, real in ((0, "double"), (1, "float"), (2, "float"), (5, "float")):
        lines += ["template __global__ void lbm::%s(lbm::StepArgs<%d>);" % (k % mode, mode) for k in STEP]
        lines += ["template __global__ void lbm::%s(lbm::StepArgs<%d>, lbm::AdjArgs<%s>);" % (k % mode, mode, real)
                  for k in REVERSE]
    src, ir = tmp_path / "kernels.hip", tmp_path / "kernels.ll"
    src.write_text("\n".join(lines) + "\n")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.hipcc()] + flags + ["-I" + os.path.join(ROOT, "paper_2608_15781_amd", "csrc"),
                                              "--cuda-device-only", "-S", "-emit-llvm", "-o", str(ir), str(src)],
                   check=True, capture_output=True)
    kernel, kernels, unset = None, set(), {}
    for line in ir.read_text().splitlines():
        if m := re.match(r"define .*amdgpu_kernel void @(\w+)", line):
            kernel = m.group(1)
            kernels.add(kernel)
        elif re.match(r"\s+%\S+ = phi .*\b(undef|poison)\b", line):
            unset[kernel] = unset.get(kernel, 0) + 1
    assert len(kernels) >= 4 * len(STEP + REVERSE)
    assert not unset, unset
