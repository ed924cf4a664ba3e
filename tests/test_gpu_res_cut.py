"""The residue contraction where the evaluation cuts the digits itself (1, 2
and 4 words, up to 32 digits; needs an MI355X): the three digit forms in the
operand orientations, with ragged rows, columns and depths (16-row blocks, 64
depths, the padding to 128), zero rows and columns, and exponents given by
the caller.

Integer arithmetic up to the one rounding, so every comparison is exact:
sampled entries against the oracle's method, and the whole output against the
slice products (the same call on a workspace too small for the planes).
"""
import numpy as np
import pytest
import torch

import mdinputs
import paper_2606_20863_amd as md
from oracle import coracle

pytestmark = pytest.mark.gpu

# m, form, M, N, K, transA, transB, leading words
CASES = [
    (1, "fp64", 1031, 515, 700, True, False, ("uniform",)),
    (2, "fp64", 255, 513, 449, False, False, ("log2uniform", 8.0)),
    (2, "fp64", 400, 272, 1025, True, True, ("uniform",)),
    (4, "fp64", 130, 143, 129, False, True, ("uniform",)),              # 30 byte planes
    (4, "int8bal", 1793, 2050, 2111, True, False, ("uniform",)),        # S odd, two-step reduction
    (4, "int8", 1801, 1999, 1985, False, True, ("log2uniform", 4.0)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"m{c[0]}-{c[1]}-{c[2]}x{c[3]}x{c[4]}")
def test_equals_oracle_and_slice_products(case):
    m, form, M, N, K, transA, transB, lead = case
    rng = np.random.Generator(np.random.PCG64(40 + m + M))
    A, B = mdinputs.mdouble(rng, m, (M, K), lead), mdinputs.mdouble(rng, m, (K, N), lead)
    A[:, M // 2, :] = 0.0
    B[:, :, N // 3] = 0.0
    A[:, 1, : K // 2] = 0.0
    dA = torch.from_numpy(np.ascontiguousarray(A.transpose(0, 2, 1)) if transA else A).cuda()
    dB = torch.from_numpy(np.ascontiguousarray(B.transpose(0, 2, 1)) if transB else B).cuda()
    opts = dict(transA=transA, transB=transB, form=form)
    _, info = md.gemm_ex(dA, dB, **opts)
    S, beta = info["S"], info["beta"]
    print(f"[res_cut] {case} S={S} beta={beta}", flush=True)
    assert md.lib().md_gemm_planes(md._FORMS[form], M, N, K, S, beta) > 0
    C, _ = md.gemm_ex(dA, dB, **opts, force_S=S, force_beta=beta)
    digit = 8 if form == "fp64" else 1
    small = (digit * S + 1) * (-(-M // 64) + -(-N // 64)) * 64 * (-(-K // 64) * 64) + (1 << 20)
    assert small < md.lib().md_gemm_workspace_size(md._FORMS[form], M, N, K, S)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    ref, _ = md.gemm_ex(dA, dB, **opts, force_S=S, force_beta=beta, workspace=ws)
    assert torch.equal(C, ref)
    rows = np.unique(np.r_[0, 1, 15, 16, M // 2, M - 1])
    cols = np.unique(np.r_[0, 17, N // 3, N - 1, min(N - 1, 255)])
    want = coracle.method_entries(A, B, beta, S, rows, cols, balanced=form == "int8bal")[3]
    np.testing.assert_array_equal(C.cpu().numpy()[:, rows][:, :, cols], want)


def test_given_exponents():
    """Exponents above the data's own (the fixed-point entry point) reach the
    cut: the integer of a depth block on the full product's grid, summed over
    the blocks, is the whole product's."""
    m, S, beta, M, N, K = 2, 5, 21, 300, 280, 1100
    rng = np.random.Generator(np.random.PCG64(9))
    A = mdinputs.mdouble(rng, m, (M, K), ("log2uniform", 6.0))
    B = mdinputs.mdouble(rng, m, (K, N), ("log2uniform", 6.0))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    assert md.lib().md_gemm_planes(0, M, N, 500, S, beta) > 0
    E, F = md.exponents(dA, dB)
    nlimb = md.fixed_limbs(beta, S, K)
    whole, scale, _ = md.gemm_fixed(dA, dB, E, F, S=S, beta=beta, form="fp64", nlimb=nlimb)
    acc = None
    for a, b in ((0, 600), (600, K)):
        X, sc, _ = md.gemm_fixed(dA[:, :, a:b], dB[:, a:b, :], E, F, S=S, beta=beta, form="fp64", nlimb=nlimb)
        assert torch.equal(sc, scale)
        acc = X if acc is None else md.fixed_add(acc, X, out=acc)
    assert torch.equal(acc, whole)
