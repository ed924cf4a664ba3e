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


def test_scratch_of_the_largest_slice_count(memory, monkeypatch):
    """A shape whose slice count changes from call to call: the scratch holds
    the planes of every count met so far."""
    n = 2048
    monkeypatch.setattr(md, "_SIZES", {})

    def sizes(S):
        return md._gemm_sizes(0, n, n, n, S)

    def call(S, force=0):
        """One call whose rule takes S; what it asked torch for."""
        opts, info = md.MDOpts(), md.MDInfo()
        opts.force_S = force
        memory.asked = []
        ws = md._auto_workspace("shape", sizes, force, "cpu", None)
        info.S = S
        md._run_with_scratch(lambda: 0, opts, ws, "shape", sizes, info)
        return memory.asked

    five, six = next(sizes(5)), next(sizes(6))
    assert five < six
    assert call(5) == []                       # nothing known: the pool
    assert call(6) == [five]
    assert call(5) == [six] and call(6) == [six] and call(5) == [six]
    # a forced count has its own size and leaves the rule's as it is
    assert call(8, force=8) == [next(sizes(8))] and call(5) == [six]
    # until the rule has run, a forced count's serves
    md._SIZES.clear()
    call(8, force=8)
    assert call(5) == [next(sizes(8))] and call(5) == [five]
    assert call(0) == [five] and call(5) == [five]   # depth 0: no slices


def test_sizes_are_bounded(memory, monkeypatch):
    monkeypatch.setattr(md, "_SIZES", {})
    for k in range(5000):
        md._note_sizes(k, 5, True, lambda S: (S, S))
    assert len(md._SIZES) <= 4096 and 4999 in md._SIZES


def test_digit_planes_lie_inside_the_panel():
    """The benchmark product: 164 residue planes of both operands, 150 planes
    of the products' residues, two units of the last diagonal's 32-bit sums
    and one magnitude plane of both operands; 27 digit planes of both are not
    added to them."""
    n = 4096
    full = md.lib().md_gemm_workspace_size(2, n, n, n, 27)
    assert md.lib().md_gemm_planes(2, n, n, n, 27, 8) == 164
    planes = 164 * 2 + 150 + 2 * 4 + 2
    assert planes * n * n < full < (planes + 1) * n * n


def test_sizes_are_worked_out_once(memory, monkeypatch):
    """Forced and hinted calls that repeat a shape do not size its scratch
    again."""
    asked = []

    class Library:
        def md_gemm_workspace_size(self, *args):
            asked.append(args)
            return 1000

    monkeypatch.setattr(md, "lib", Library)
    md._gemm_size.cache_clear()
    for _ in range(3):
        md._auto_workspace("shape", lambda S: md._gemm_sizes(0, 64, 64, 64, S), 5, "cpu", None)
    md._gemm_size.cache_clear()
    assert len(asked) == 1 and memory.asked == [1000] * 3


def test_the_depth_is_cut_into_parts():
    """The products of test_gpu_parts.py: what their scratch takes beyond the
    least is two parts' integers and scales or more."""
    from test_gpu_parts import CASES
    for m, form, M, N, K in CASES:
        for G in (4, 8, 16):
            beta, S, _, _ = md.choose_params(form, K, 50 * m, G)
            full, least = md._gemm_sizes(md._FORMS[form], M, N, K, S)
            assert md.lib().md_gemm_planes(md._FORMS[form], M, N, K, S, beta) == 0
            words, rest = divmod(full - least - 256, 4 * M * N)
            parts, one = divmod(words, md.fixed_limbs(beta, S, K))
            assert rest == 0 and one == 1 and 2 <= parts <= 64, (m, form, M, N, K, S)
