"""Products on workspaces of different sizes (needs an MI355X): the size that
the fastest way takes, the least one, and one byte less than the fastest way
takes give the same words, for products that run the residue contraction, the
depth parts, the bands with their sum buffer and the FP64 slices.
"""
import numpy as np
import pytest
import torch

import mdinputs
import paper_2606_20863_amd as md

pytestmark = pytest.mark.gpu

# m, form, M, N, K, whether more than the least is of use
CASES = [
    (8, "int8bal", 300, 513, 640, True),      # residues, digit planes apart
    (2, "fp64", 513, 700, 640, True),         # residues, digits cut on the way
    (4, "int8", 700, 24, 1500, True),         # depth parts
    (16, "int8bal", 16, 24, 24, False),       # bands
    (4, "fp64", 64, 80, 64, False),           # FP64 slices
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"m{c[0]}-{c[1]}-{c[2]}x{c[3]}x{c[4]}")
def test_same_words_on_every_size(case):
    m, form, M, N, K, more = case
    rng = np.random.Generator(np.random.PCG64(M + K))
    dA = torch.from_numpy(mdinputs.mdouble(rng, m, (M, K), ("uniform",))).cuda()
    dB = torch.from_numpy(mdinputs.mdouble(rng, m, (K, N), ("uniform",))).cuda()
    want, info = md.gemm_ex(dA, dB, form=form)
    S, beta = info["S"], info["beta"]
    full, least = md._gemm_sizes(md._FORMS[form], M, N, K, S)
    assert (full > least) == more
    for size in (full, least, max(least, full - 4097)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        C, _ = md.gemm_ex(dA, dB, form=form, force_S=S, force_beta=beta, workspace=ws)
        assert torch.equal(C, want), size
        C, _ = md.gemm_ex(dA, dB, form=form, workspace=ws)
        assert torch.equal(C, want), size


def test_slice_count_changes_from_call_to_call():
    """One shape through gemm with data of two spans by turns: the words of
    the pool's calls every time."""
    m, M, N, K = 2, 640, 520, 700
    rng = np.random.Generator(np.random.PCG64(11))
    A = torch.from_numpy(mdinputs.mdouble(rng, m, (M, K), ("uniform",))).cuda()
    B = torch.from_numpy(mdinputs.mdouble(rng, m, (K, N), ("uniform",))).cuda()
    small, even = A.clone(), B.clone()
    small[:, :, ::2] *= 2.0 ** -24         # every other depth far below the rows' exponents,
    even[:, 1::2] = 0.0                    # and the columns meet those depths alone
    cases = [(A, B), (small, even)]
    want = [md.gemm_ex(a, b, pool=True) for a, b in cases]
    assert len({i["S"] for _, i in want}) > 1
    for _ in range(3):
        for (a, b), (C, _) in zip(cases, want):
            assert torch.equal(md.gemm(a, b), C)


def test_pool_gives_large_scratch_back():
    """A product on the library's pool whose planes take more than 4 GiB:
    with the call ended, no more than that stays taken from the device."""
    m, n, S = 4, 4096, 27
    assert next(md._gemm_sizes(2, n, n, n, S)) > 6 << 30
    gen = torch.Generator(device="cuda").manual_seed(3)
    A = torch.rand((m, n, n), generator=gen, dtype=torch.float64, device="cuda") - 0.5
    A *= 2.0 ** (-54 * torch.arange(m, device="cuda", dtype=torch.float64))[:, None, None]
    C = torch.empty_like(A)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    md.gemm_ex(A, A.clone(), C, form="int8bal", force_S=S, force_beta=8, pool=True)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] <= (4 << 30) + (64 << 20)
