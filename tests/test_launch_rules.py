"""Host rules of the launchers (csrc/launch_rules.h), compiled by themselves."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GRID_BLOCKS = (2 ** 32 - 1) // 256  # of 256 threads, in one dimension of a grid


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule(expr, ...): the values of C++ integer expressions over the header's rules."""
    d = tmp_path_factory.mktemp("rules")

    def run(*exprs):
        src, exe = d / "r.cpp", d / "r"
        body = "".join(f'printf("%lld\\n", (long long)({e}));' for e in exprs)
        src.write_text('#include <cstdio>\n#include "launch_rules.h"\nusing namespace lbm;\n'
                       f"int main() {{{body}}}\n")
        subprocess.run(["g++", "-std=c++17", "-I",
                        os.path.join(ROOT, "paper_2505_10171_amd", "csrc"), str(src), "-o",
                        str(exe)], check=True)
        return [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True,
                                               text=True).stdout.split()]
    return run


@pytest.mark.parametrize("nodes,rows,R,r", [
    (32 ** 3, 1, 4, 4), (512 * 256 * 192, 500, 4, 4), (256 ** 3, 4096, 10, 10),
    # grids beyond one dimension with a node per thread
    (240 ** 3, 501, 102, 3), (256 ** 3, 1281, 80, 10), (226 * 10 ** 6, 4096, 60, 60)])
def test_capillary_blocks_fit_the_grid(rule, nodes, rows, R, r):
    """Those of all particles, one of radius R and the others r, share a flat grid with
    the fluid's."""
    fluid, own = -(-nodes // 256), f"box_blocks({2 * R + 4}) + {rows - 1} * box_blocks({2 * r + 4})"
    per, = rule(f"particle_blocks_flat({fluid}, {rows}, {2 * R + 3}, {own})")
    assert 1 <= per <= -(-(2 * R + 3) ** 3 // 256) and fluid + rows * per <= GRID_BLOCKS


def test_where_a_kernel_stores_directly(rule):
    """Only into memory of the workspace's own GPU; -1: not device memory, or unknown."""
    got = rule("stores_directly(true, 0, 0)", "stores_directly(true, 1, 1)",
               "stores_directly(true, 1, 0)", "stores_directly(true, 0, 1)",
               "stores_directly(false, -1, 0)", "stores_directly(false, -1, -1)",
               "stores_directly(false, 0, 0)", "stores_directly(true, 0, -1)")
    assert got == [1, 1, 0, 0, 0, 0, 0, 0]


@pytest.mark.parametrize("rows,R,r", [
    (1, 4, 4), (500, 4, 4), (1, 100, 100), (4096, 10, 10), (500, 12, 12), (401, 20, 3),
    (512, 14, 2), (60000, 30, 1)])
def test_particle_blocks(rule, rows, R, r):
    """A node per thread where the boxes are alike, a bounded grid where one is far
    larger than the others."""
    full = -(-(2 * R + 4) ** 3 // 256)
    own = full + (rows - 1) * -(-(2 * r + 4) ** 3 // 256)
    per, = rule(f"particle_blocks({rows}, {2 * R + 4}, {own})")
    if R == r or rows * full <= 32768:
        assert per == full
    else:
        assert per == max(1, 32768 // rows)
