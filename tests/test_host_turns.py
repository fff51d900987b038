"""How a launch deals its blocks out to the XCDs, compiled for the host from the library's own header: for any number of
blocks that a bounce needs, none included, and any larger grid, the workgroups work as every block exactly once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r'''
#include "trace_core.h"
#include <cstdio>
#include <vector>

int main() {
    long bad = 0, n = 0;
    const uint32_t most[] = {1, 7, 8, 9, 2047, 2048, 2049, 4096, 20000, 65536};
    for (uint32_t m : most) {
        const uint32_t groups = pcrl::xcd_groups(m);
        for (uint32_t blocks = 0; blocks <= m; blocks += m > 4096 ? 61 : 1, ++n) {
            std::vector<unsigned char> seen(blocks, 0);
            for (uint32_t g = 0; g < groups; ++g) {
                const uint32_t b = pcrl::xcd_turn(blocks, g);
                if (b < blocks) bad += seen[b]++ != 0;
            }
            for (unsigned char s : seen) bad += s != 1;
        }
    }
    std::printf("checked %ld bad %ld\\n", n, bad);
    return bad != 0;
}
'''


def test_every_block_once(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "turns.hip", tmp_path / "turns"
    src.write_text(HARNESS)
    subprocess.run([hipcc, "--offload-host-only", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2402_13747_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "bad 0" in r.stdout, (r.returncode, r.stdout[-2000:])
