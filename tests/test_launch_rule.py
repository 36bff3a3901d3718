"""Host-side rules of the launches (no GPU): the default block against the LDS
that a mechanism's compaction slots take."""
import subprocess

from paper_2506_02602_amd import build, codegen

PROGRAM = r"""
#include <cstdio>
#include "launch.h"
int main() {
  for (int ns = 1; ns <= 64; ++ns)
    printf("%d %d %d %zu\n", chemgpu::size_block(ns, false), chemgpu::size_block(ns, true),
           chemgpu::fit_block(ns, 128), chemgpu::slot_bytes(ns, 1));
}
"""


def test_default_blocks_fit_every_mechanism(tmp_path):
    """A call that names no block is accepted for 1 to 64 species, whatever the
    number of reactions (which decides how many lanes a cell takes in the
    cooperative kernel): the default block's slots fit 64 KB, and it is cut
    only where it has to be."""
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    rows = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    seen = set()
    for ns in range(1, 65):
        narrow, wide, other, lane = map(int, rows[ns - 1].split())
        assert lane == (ns + 4) * 8 + 24
        for nr in (1, ns, 32, 33, 64, 200):
            g = codegen.coop_group(dict(species=[0] * ns, reactions=[0] * nr))
            block = wide if 64 // g == 1 else narrow
            want = 128 if 64 // g == 1 else 256
            assert block * lane <= 65536 and block % 64 == 0
            assert block == want or 2 * block * lane > 65536
            seen.add((ns, nr, block))
        assert other * lane <= 65536 and (other == 128 or 2 * other * lane > 65536)
    assert (25, 32, 256) in seen and (26, 32, 128) in seen and (32, 32, 128) in seen
