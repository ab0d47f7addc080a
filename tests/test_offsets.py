"""The rule that chooses 32- or 64-bit array offsets (csrc/offsets.hpp, compiled here as host code), against the
byte offsets that the kernels form, at plane strides on both sides of every limit. CPU only."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STORAGES = {"fp64": (8, 8), "fp32": (4, 4), "fp16": (2, 4), "bf16": (2, 4)}  # bytes stored, bytes of the arithmetic type
LIMIT = 1 << 32

DRIVER = r"""
#include <cstdio>
#include "offsets.hpp"
int main() {
  size_t N, ps, s, r;
  while (std::scanf("%zu %zu %zu %zu", &N, &ps, &s, &r) == 4)
    std::printf("%d %d\n", int(lbm::wide(lbm::step_offsets(N, ps, s, r))), int(lbm::wide(lbm::adjoint_offsets(N, ps, s, r))));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("offsets")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2608_15781_amd", "csrc"), "-o",
                    str(d / "driver"), str(d / "driver.cpp")], check=True)

    def ask(rows):
        out = subprocess.run([str(d / "driver")], input="\n".join("%d %d %d %d" % r for r in rows), text=True,
                             capture_output=True, check=True).stdout
        return [tuple(bool(int(v)) for v in line.split()) for line in out.splitlines()]

    return ask


def _pair_distance():
    """The largest distance of two planes of opposite directions, from the velocities themselves."""
    M = np.loadtxt(os.path.join(ROOT, "tests", "golden", "d3q19_matrix_M.txt"), dtype=int)
    c = [tuple(v) for v in M.T]  # (x, y, z) of every direction
    return max(abs(c.index(tuple(-x for x in v)) - i) for i, v in enumerate(c))


def _largest_offsets(N, ps, s, r):
    """Last byte that each family of accesses reaches from its base: (forward kernels, reverse kernels). A
    pair's upper plane is addressed from the lower plane's base."""
    pair = _pair_distance()
    last = lambda element, size: element * size + size - 1
    forward = dict(populations=last(pair * ps + ps - 1, s), vectors=last(ps - 1, 4 * r), pairs=last(N - 1, 2 * r),
                   lists=last(N - 1, 8), species_totals=last(ps - 1, r))
    reverse = dict(forward, adjoint_populations=last(pair * ps + ps - 1, r), adjoint_vectors=last(ps - 1, 4 * r))
    return max(forward.values()), max(reverse.values())


@pytest.mark.parametrize("storage", sorted(STORAGES))
@pytest.mark.parametrize("porosity", [1.0, 0.45])
def test_narrow_offsets_stay_below_four_gigabytes(rule, storage, porosity):
    s, r = STORAGES[storage]
    unit = 256 // s
    rows = []
    for per_entry in (1, 2, 4, 8, 16, 6 * s, 6 * r, 4 * r, 2 * r):  # strides round every multiple's limit
        for step in (-3, -1, 0, 1, 3):
            ps = (LIMIT // per_entry // unit + step) * unit
            N = int(ps / porosity)
            if 0 < ps <= N < 2 ** 31:
                rows.append((N, ps, s, r))
    assert rows
    for row, (step_wide, adjoint_wide) in zip(rows, rule(rows)):
        forward, reverse = _largest_offsets(*row)
        assert step_wide or forward < LIMIT, (row, forward)
        assert adjoint_wide or reverse < LIMIT, (row, reverse)
        # wide only where it is needed (to the granularity of the plane stride)
        slack = 64 * unit * r
        assert not step_wide or forward + slack >= LIMIT, (row, forward)
        assert not adjoint_wide or reverse + slack >= LIMIT, (row, reverse)


@pytest.mark.parametrize("storage", ["fp16", "bf16"])
def test_reverse_pass_of_two_byte_storages_goes_wide_first(rule, storage):
    """600^3 without solids: the step's offsets fit 32 bits, the adjoint populations' do not."""
    s, r = STORAGES[storage]
    N = 600 ** 3
    forward, reverse = _largest_offsets(N, N, s, r)
    assert forward < LIMIT < reverse
    assert rule([(N, N, s, r)]) == [(False, True)]
