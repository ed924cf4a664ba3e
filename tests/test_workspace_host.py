"""The scratch of a product (host only): sizing calls with no slices return
the statistics and magnitude planes, in a process of their own (a division by
the slice count would end it), and a call for which the device has no room
takes less."""
import subprocess
import sys

import pytest
import torch

import paper_2606_20863_amd as md


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


@pytest.fixture
def memory(monkeypatch):
    """torch.empty with room for ``memory.room`` bytes; ``memory.asked``
    lists what it was asked for."""
    class Memory:
        room, asked = 1 << 62, []

        def empty(self, n, **kw):
            self.asked.append(n)
            if n > self.room:
                raise torch.OutOfMemoryError("no room")
            return torch.ones(0, dtype=torch.uint8)

    mem = Memory()
    mem.asked = []
    monkeypatch.setattr(md.torch, "empty", mem.empty)
    return mem


def test_less_scratch_where_memory_is_short(memory):
    """The benchmark product (9 GB of residue planes): with room for the
    planes, for the slice products (1 GB) and for neither."""
    n, S = 4096, 27
    full, least = md._gemm_sizes(2, n, n, n, S)
    assert least <= md.lib().md_gemm_workspace_size(2, n, n, n, S) == full
    # digits and magnitudes of both operands, and less than a percent more
    assert 2 * 28 * n * n < least < 2.02 * 28 * n * n < full / 4

    def ask(room):
        memory.room, memory.asked = room, []
        return md._auto_workspace("shape", lambda s: md._gemm_sizes(2, n, n, n, s), S, "cpu", None)

    assert ask(full) is not None and memory.asked == [full]
    assert ask(full - 1) is not None and memory.asked == [full, least]
    assert ask(least - 1) is None and memory.asked == [full, least]   # the library's pool


@pytest.mark.parametrize("form,M,N,K,S", [(2, 4096, 24, 4096, 27), (0, 64, 64, 64, 5), (1, 300, 200, 100, 105),
                                          (0, 1024, 1024, 1024, 40), (2, 1024, 1024, 1024, 56)])
def test_least_is_not_above_the_size(form, M, N, K, S):
    full, least = md._gemm_sizes(form, M, N, K, S)
    assert 0 < least <= full
