"""The one-launch exponent pass and magnitude split (needs an MI355X): shared
exponents (the debug dump) and the slice rule's statistics at the edges of its
blocks (16 rows; 64, 256, 512, 1024 and 2048 depths) in all orientations, with
zero rows, subnormal and power-of-two leading words.  Integers, so exact: the
exponents against the oracle's, the ratio and span exponents against the same
data padded with zero columns to a depth that takes the separate passes.
"""
import numpy as np
import pytest
import torch

import paper_2606_20863_amd as md
from oracle import exact as ox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 63, 64, 65, 255, 257, 513, 1024, 1025, 2048])
@pytest.mark.parametrize("transA,transB", [(False, False), (True, True)])
def test_exponents_and_statistics(K, transA, transB):
    rng = np.random.Generator(np.random.PCG64(K))
    M, N = 33, 18
    A = np.exp2(rng.uniform(-3, 3, (1, M, K))) * rng.choice([-1.0, 1.0], (1, M, K))
    B = np.exp2(rng.uniform(-3, 3, (1, K, N)))
    A[0, 5] = 0.0
    A[0, 7] = 2.0 ** rng.integers(-4, 4, K)
    B[0, :, 2] = 2.0 ** -1060 * (1 + rng.integers(0, 3, K))

    def call(a, b):
        dbg = {"E": torch.zeros(M, dtype=torch.int32, device="cuda"), "F": torch.zeros(N, dtype=torch.int32, device="cuda")}
        ta = torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 1) if transA else a)).cuda()
        tb = torch.from_numpy(np.ascontiguousarray(b.transpose(0, 2, 1) if transB else b)).cuda()
        _, info = md.gemm_ex(ta, tb, transA=transA, transB=transB, form="int8bal", debug=dbg)
        return dbg["E"].cpu().numpy(), dbg["F"].cpu().numpy(), info

    E, F, info = call(A, B)
    np.testing.assert_array_equal(E, ox.row_exponents(A[0])[0])
    np.testing.assert_array_equal(F, ox.row_exponents(B[0].T)[0])
    pad = 2304 - K
    E2, F2, info2 = call(np.concatenate([A, np.zeros((1, M, pad))], 2), np.concatenate([B, np.zeros((1, pad, N))], 1))
    np.testing.assert_array_equal(E, E2)
    np.testing.assert_array_equal(F, F2)
    for key in ("span_A", "span_B", "G_span", "input_flags"):
        assert info[key] == info2[key], key

    # the magnitude product, without the zero row and the subnormal column
    keep = np.r_[0:5, 6:M]
    A2, B2 = A[:, keep], np.delete(B, 2, 2)
    q = np.floor(np.abs(A2[0]) * 2.0 ** (7 - np.array(ox.row_exponents(A2[0])[0], dtype=float))[:, None])
    p = np.floor(np.abs(B2[0]) * 2.0 ** (7 - np.array(ox.row_exponents(B2[0].T)[0], dtype=float))[None])
    least = int((q.astype(np.int64) @ p.astype(np.int64)).min())
    M, N = A2.shape[1], B2.shape[2]
    _, _, info = call(A2, B2)
    g = 0
    while least << g < (K << 14) + 1:
        g += 1
    assert info["G_rho"] == g
