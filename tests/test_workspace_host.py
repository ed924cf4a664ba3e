"""The scratch sizes (host only): sizing calls with no slices return the slice
products' statistics and magnitude planes, in a process of their own (a
division by the slice count would end it)."""
import subprocess
import sys

import pytest


@pytest.mark.parametrize("form", [0, 1, 2])
def test_size_without_slices(form):
    code = ("import paper_2606_20863_amd as md\n"
            f"print(*[md.lib().md_gemm_workspace_size({form}, n, n, n, 0) for n in (64, 1000, 4096)])")
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert res.returncode == 0, res
    # six int32 arrays of n + 64 entries, 64 words of statistics and the
    # alignment of nine arrays, 4096 to spare; two planes of one byte an entry
    pad = {64: (64, 64), 1000: (1024, 1024), 4096: (4096, 4096)}
    want = [(6 * ((n + 64 + 63) // 64 * 64) + 64) * 4 + 7 * 256 + 4096 + 2 * pad[n][0] * pad[n][1] for n in pad]
    assert [int(x) for x in res.stdout.split()] == want
