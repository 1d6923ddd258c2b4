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


@pytest.mark.parametrize("nodes,rows,R", [
    (32 ** 3, 1, 4), (512 * 256 * 192, 500, 4), (256 ** 3, 4096, 10),
    # grids beyond one dimension with a node per thread
    (240 ** 3, 501, 102), (256 ** 3, 1281, 80), (226 * 10 ** 6, 4096, 60)])
def test_capillary_blocks_fit_the_grid(rule, nodes, rows, R):
    side, fluid = 2 * R + 3, -(-nodes // 256)
    per, = rule(f"capillary_blocks({fluid}, {rows}, {side})")
    full = -(-side ** 3 // 256)
    assert 1 <= per <= full and fluid + rows * per <= GRID_BLOCKS
    # a node per thread wherever that fits
    assert per == full or fluid + rows * (per + 1) > GRID_BLOCKS


def test_where_a_kernel_stores_directly(rule):
    """Only into memory of the workspace's own GPU; -1: not device memory, or unknown."""
    got = rule("stores_directly(true, 0, 0)", "stores_directly(true, 1, 1)",
               "stores_directly(true, 1, 0)", "stores_directly(true, 0, 1)",
               "stores_directly(false, -1, 0)", "stores_directly(false, -1, -1)",
               "stores_directly(false, 0, 0)", "stores_directly(true, 0, -1)")
    assert got == [1, 1, 0, 0, 0, 0, 0, 0]


@pytest.mark.parametrize("rows,R", [(1, 4), (500, 4), (1, 100), (401, 20), (4096, 10), (60000, 3)])
def test_particle_blocks(rule, rows, R):
    side = 2 * R + 4
    per, = rule(f"particle_blocks({rows}, {side})")
    full = -(-side ** 3 // 256)
    assert 1 <= per <= full
    assert per == 1 or rows * per <= 32768
    assert per == full or rows * (per + 1) > 32768
