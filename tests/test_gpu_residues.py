"""The residue contraction on the GPU (needs an MI355X): sizes where the
library takes it in place of the slice products, at the edges of its tiles
(256 outputs, 16-row blocks, 64 and 128 depths), in the three forms, with
odd and even slice counts, one and two tiles of coefficients, sums that need
the two-step reduction, several units on the last diagonal and several
panels.

It is integer arithmetic up to the one rounding, so every comparison is
exact: sampled entries against the oracle's method, and the whole output
against the same call on a workspace too small for the residue planes, which
runs the slice products.
"""
import numpy as np
import pytest
import torch

import mdinputs
import paper_2606_20863_amd as md
from oracle import coracle
from oracle import exact as ox

pytestmark = pytest.mark.gpu

# m, form, M, N, K, transA, transB, leading words
CASES = [
    (16, "int8bal", 129, 257, 193, False, False, ("log2uniform", 6.0)),   # S odd, two coefficient tiles twice
    (16, "int8", 256, 240, 130, True, False, ("uniform",)),               # S even
    (8, "int8bal", 300, 513, 640, False, True, ("log2uniform", 16.0)),
    (8, "int8", 257, 255, 1000, True, True, ("uniform",)),
    (4, "int8bal", 256, 250, 4097, False, False, ("uniform",)),           # two-step reduction
    (4, "fp64", 255, 257, 320, False, True, ("log2uniform", 8.0)),        # three bytes per digit
    (2, "fp64", 513, 700, 2049, True, False, ("uniform",)),               # small L, two-step reduction
    (1, "fp64", 1100, 1030, 777, False, False, ("uniform",)),             # two bytes or three, L = 3
    (16, "fp64", 129, 300, 65, False, False, ("log2uniform", 4.0)),
]


def operands(case, seed):
    m, form, M, N, K, transA, transB, lead = case
    rng = np.random.Generator(np.random.PCG64(seed))
    A = mdinputs.mdouble(rng, m, (M, K), lead)
    B = mdinputs.mdouble(rng, m, (K, N), lead)
    A[:, M // 2, :] = 0.0
    B[:, :, N // 3] = 0.0
    dA = torch.from_numpy(np.ascontiguousarray(A.transpose(0, 2, 1)) if transA else A).cuda()
    dB = torch.from_numpy(np.ascontiguousarray(B.transpose(0, 2, 1)) if transB else B).cuda()
    return A, B, dA, dB


def slice_workspace(form, S, M, N, K):
    """Bytes that hold the slice products' scratch (digit planes, statistics,
    the diagonal sums of the banded kernels)."""
    Mp, Np, Kp = -(-M // 64) * 64, -(-N // 64) * 64, -(-K // 64) * 64
    digit = 8 if form == "fp64" else 1
    return (digit * S + 1) * (Mp + Np) * Kp + 8 * S * Mp * Np + (1 << 20)


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"m{c[0]}-{c[1]}-{c[2]}x{c[3]}x{c[4]}")
def test_equals_oracle_and_slice_products(case):
    m, form, M, N, K, transA, transB, _ = case
    A, B, dA, dB = operands(case, 300 + m + M)
    opts = dict(transA=transA, transB=transB, form=form)
    _, info = md.gemm_ex(dA, dB, **opts)
    S, beta = info["S"], info["beta"]
    print(f"[residues] {case} S={S} beta={beta}", flush=True)
    need = md.lib().md_gemm_workspace_size(md._FORMS[form], M, N, K, S)
    small = slice_workspace(form, S, M, N, K)
    assert need > small, "the library does not take the residue contraction here"
    C, _ = md.gemm_ex(dA, dB, **opts, force_S=S, force_beta=beta)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    ref, _ = md.gemm_ex(dA, dB, **opts, force_S=S, force_beta=beta, workspace=ws)
    assert torch.equal(C, ref)
    rows = np.unique(np.r_[0, 15, 16, M // 2, M - 1, min(M - 1, 128)])
    cols = np.unique(np.r_[0, 17, N // 3, N - 1, min(N - 1, 255)])
    want = coracle.method_entries(A, B, beta, S, rows, cols, balanced=form == "int8bal")[3]
    np.testing.assert_array_equal(C.cpu().numpy()[:, rows][:, :, cols], want)


def test_fixed_point_integers():
    """md_gemm_fixed through the residues: sampled integers and scales equal
    the oracle's, with limbs past the fold's own."""
    m, S, beta, K = 8, 52, 8, 512
    A, B, dA, dB = operands((m, "int8bal", 280, 300, K, False, False, ("log2uniform", 8.0)), 7)
    nlimb = md.fixed_limbs(beta, S, K) + 4
    X, scale, _ = md.gemm_fixed(dA, dB, S=S, beta=beta, form="int8bal", nlimb=nlimb)
    rows, cols = [0, 17, 140, 279], [1, 100, 255, 299]
    Xo, so = ox.fixed_product(A[:, rows], B[:, :, cols], beta, S, balanced=True)
    got = X.cpu().numpy().view(np.uint32)[:, rows][:, :, cols].astype(object)
    got = sum(got[k] << (32 * k) for k in range(nlimb))
    got = np.where(got >= 1 << (32 * nlimb - 1), got - (1 << (32 * nlimb)), got)
    assert np.array_equal(got, Xo)
    assert np.array_equal(scale.cpu().numpy()[rows][:, cols], so)


def test_several_panels():
    """Outputs that do not fit one panel of residue planes."""
    m, form, M, N, K = 2, "fp64", 11800, 11700, 512
    gen = torch.Generator(device="cuda").manual_seed(5)
    dA = torch.rand((m, M, K), generator=gen, dtype=torch.float64, device="cuda") - 0.5
    dB = torch.rand((m, K, N), generator=gen, dtype=torch.float64, device="cuda") - 0.5
    dA[1] *= 2.0 ** -60
    dB[1] *= 2.0 ** -60
    C, info = md.gemm_ex(dA, dB, form=form)
    rows = np.r_[0, 5903, 5904, 8000, M - 1]
    cols = np.r_[0, 5850, 5888, 9001, N - 1]
    A, B = dA[:, rows].cpu().numpy(), dB[:, :, cols].cpu().numpy()
    want = coracle.method_entries(A, B, info["beta"], info["S"], np.arange(5), np.arange(5))[3]
    np.testing.assert_array_equal(C[:, rows][:, :, cols].cpu().numpy(), want)
