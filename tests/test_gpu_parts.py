"""INT8 products whose depth is cut into parts that run side by side (few
output tiles, or a depth over several exactness chunks; needs an MI355X):
sampled entries against the oracle's method, and every word against the same
call on a workspace that holds no parts.  Integer sums, so exact.
"""
import numpy as np
import pytest
import torch

import mdinputs
import paper_2606_20863_amd as md
from oracle import coracle

pytestmark = pytest.mark.gpu

# m, form, M, N, K
CASES = [
    (4, "int8bal", 700, 24, 1500),     # one tile column, a last part shorter than the others
    (4, "int8", 1, 1, 3000),           # one output
    (4, "int8bal", 65, 33, 9001),      # more than one exactness chunk (two at least)
    (2, "int8bal", 64, 32, 4096),
    (2, "int8", 130, 100, 2049),
    (1, "int8bal", 40, 70, 20000),     # few slices, deep
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"m{c[0]}-{c[1]}-{c[2]}x{c[3]}x{c[4]}")
def test_parts(case):
    m, form, M, N, K = case
    rng = np.random.Generator(np.random.PCG64(K))
    A = mdinputs.mdouble(rng, m, (M, K), ("log2uniform", 3.0))
    B = mdinputs.mdouble(rng, m, (K, N), ("uniform",))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    _, info = md.gemm_ex(dA, dB, form=form)
    S, beta = info["S"], info["beta"]
    Mp, Np, Kp = -(-M // 32) * 32, -(-N // 32) * 32, -(-K // 64) * 64
    whole = (S + 1) * (Mp + Np) * Kp + (1 << 15)   # digit and magnitude planes, statistics
    need = md.lib().md_gemm_workspace_size(md._FORMS[form], M, N, K, S)
    nlimb = md.fixed_limbs(beta, S, K)
    assert need > whole - (1 << 15) + 2 * 4 * nlimb * M * N, "the library does not cut the depth here"
    C, _ = md.gemm_ex(dA, dB, form=form, force_S=S, force_beta=beta)
    ws = torch.empty((S + 0) * (Mp + Np) * Kp + 4 * (3 * (M + N) + 512) + 4096, dtype=torch.uint8, device="cuda")
    ref, _ = md.gemm_ex(dA, dB, form=form, force_S=S, force_beta=beta, workspace=ws)
    assert torch.equal(C, ref)
    rows = np.unique(np.r_[0, M // 2, M - 1])
    cols = np.unique(np.r_[0, N // 2, N - 1])
    want = coracle.method_entries(A, B, beta, S, rows, cols, balanced=form == "int8bal")[3]
    np.testing.assert_array_equal(C.cpu().numpy()[:, rows][:, :, cols], want)
