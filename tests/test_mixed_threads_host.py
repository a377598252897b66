"""Threads of the mixed-radix launches (pss_kernels.h), on the host: whole waves
that hold the block's elements, and, in launches too small to fill the chip, a
thread for each element up to 256, as every such launch had before the blocks
went by size (with fewer, 250 sites of KPZ took 13.8 us a step instead of 7.5)."""

import os
import subprocess

import pytest

from paper_2405_02410_amd import build as b

PROGRAM = r"""
#include <cstdio>
#include "pss_kernels.h"
int main() {
    for (int N = 2; N <= 4096; N += 2) {
        pss::MrPlan mr{};
        if (!pss::mr_plan(N, &mr)) continue;
        for (int tc = 1; tc <= 2; ++tc)
            for (unsigned blocks : {1u, 100u, 1024u, 1025u, 6000u})
                std::printf("%d %u %d %d\n", tc * N, blocks, pss::mr_threads(tc * N), pss::mr_block_threads(tc * N, blocks));
    }
}
"""


def test_threads_of_the_mixed_radix_launches(tmp_path):
    try:
        hipcc = b._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src = tmp_path / "threads.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "threads"
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-w", "-I", b.CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=300, env=dict(os.environ))
    rows = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(rows) > 500
    for row in rows:
        n, blocks, few, t = (int(v) for v in row.split())
        assert t % 64 == 0 and 64 <= few <= t <= 1024
        assert t >= min(n, 256) if blocks <= 1024 else t == few
        assert t == few or t <= 256
