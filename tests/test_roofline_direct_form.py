"""Host checks of the work that the bench's smoother rates are rates of: the form
that runs, not the one in which the step is stated."""
import itertools
import os
import re
import subprocess

import pytest

from paper_2405_18982_amd import roofline

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rules_are_the_kernels(tmp_path):
    """takes_direct_form against the rules the kernels are compiled with."""
    src = tmp_path / "rules.cpp"
    src.write_text("""
#include "dgmg_internal.h"
#include <cstdio>
int main() {
  for (int d = 2; d <= 3; ++d)
    for (int k = 1; k <= 7; ++k)
      for (int s = 4; s <= 8; s += 4)
        for (int N = 4; N <= 1024; N *= 2)
          std::printf("%d %d %d %d %d\\n", d, k, s, N,
                      dgmg::direct_smoother(d, k) && N < dgmg::direct_below(d, k, s));
}
""")
    exe = tmp_path / "rules"
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_18982_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True, timeout=100)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=20).stdout
    rows = [tuple(map(int, ln.split())) for ln in out.splitlines()]
    assert len(rows) == 2 * 7 * 2 * 9
    for d, k, s, N, direct in rows:
        assert roofline.takes_direct_form(d, k, N, s) == bool(direct), (d, k, s, N)


@pytest.mark.parametrize("dim,k,N,colour", [(2, 5, 8, 0), (3, 3, 4, 0), (3, 3, 8, 7), (3, 2, 6, 5)])
def test_direct_bytes_by_nodes(dim, k, N, colour):
    """Per patch, node by node: b and the written x on V_j, x elsewhere on the tile."""
    E, total = 2 * (k + 1), 0
    for lo in itertools.product(*roofline.patch_los(N, colour, dim)):
        for node in itertools.product(range(E), repeat=dim):
            dropped = any((p == 0 and l > 0) or (p == E - 1 and l + 2 < N) for p, l in zip(node, lo))
            total += 1 if dropped else 2
    assert roofline.direct_colour_counts(dim, k, N, colour)["bytes"] == 8 * total


def test_flops_are_below_the_counted_instructions():
    """3-D Q7 64^3 FP64: the counter passes show the fused multiply-adds a wave of the
    smoother executes (four waves a patch, 64 lanes); they include the lines of dropped
    nodes, a quarter of all, and no more than that."""
    text = open(os.path.join(ROOT, "profiles", "k_smooth_poisson3d_q7_64c_counters.txt")).read()
    # the colour of the fewest patches: most of them interior
    m = re.findall(r"k_smooth<double, 1, 1,[^>]*> grid=(\d+) .*?SQ_INSTS_VALU_FMA_F64\s+\S+\s+per wave\s+(\S+)", text,
                   re.S)
    grid, fma = min((int(g), float(f)) for g, f in m)
    patches = 31 ** 3
    assert grid == 256 * patches
    executed = 2 * fma * 4 * 64 * patches
    counted = roofline.direct_colour_counts(3, 7, 64, 7)["flops"]
    assert 0.7 * executed <= counted <= executed
    # the step as stated is more than twice that
    assert roofline.smooth_colour_counts(3, 7, 64, 7)["flops"] > 2 * counted


def test_run_counts_follow_the_form():
    assert roofline.smooth_run_counts(2, 3, 16) == roofline.smooth_step_counts(2, 3, 16)
    assert roofline.smooth_run_counts(2, 4, 128, s=4) == roofline.smooth_step_counts(2, 4, 128, s=4)
    tot = [roofline.direct_colour_counts(3, 3, 8, c, nrhs=2) for c in range(8)]
    run = roofline.smooth_run_counts(3, 3, 8, nrhs=2)
    assert run == {key: sum(t[key] for t in tot) for key in ("bytes", "flops")}
