"""The residue contraction at the ends of its ranges (needs an MI355X): 65,536
depths, the most that it takes, and 65,537; 2,048 depths, the most of the
one-step reduction, and 2,049; more than 128 digit bytes an entry; INT8 digits
of one and two words.

Operands whose sums come near the bounds with one sign: entries all alike,
drawn so that at one point the residues modulo 251 of both operands are +-125,
and entries of the largest digits (balanced ones all -128 below the first).
Integer arithmetic up to the one rounding, so every comparison is exact: the
whole output against the slice products (the same call on a workspace that
holds no planes), sampled entries against the oracle's method.
"""
import random

import numpy as np
import pytest
import torch

import mdinputs
import paper_2606_20863_amd as md
from oracle import coracle

pytestmark = pytest.mark.gpu


def value_at(digits, x, beta, form, second, p):
    """The operand's polynomial of digits at x modulo p."""
    if form == "fp64":
        blocks = digits
    else:
        S = len(digits)
        shift = [0] if second and S % 2 == 0 else []
        d = shift + list(digits)
        blocks = [(d[2 * c] << beta) + d[2 * c + 1] for c in range(S // 2)]
    return sum(b * pow(x, c, p) for c, b in enumerate(blocks)) % p


def draw_digits(rng, S, beta, form):
    if form == "int8bal":
        return [rng.randint(33, 62)] + [rng.randint(-128, 127) for _ in range(S - 1)]
    return [rng.randint(1 << (beta - 1), (1 << beta) - 1)] + [rng.randint(0, (1 << beta) - 1) for _ in range(S - 1)]


def largest_digits(S, beta, form):
    if form == "int8bal":
        return [62] + [-128] * (S - 1)
    return [(1 << beta) - 1] * S


def words(digits, m, beta, form):
    """The entry with these digits and shared exponent 0: words of 53 bits."""
    S = len(digits)
    X = sum(d << (beta * (S - 1 - s)) for s, d in enumerate(digits))
    bits = beta * S - (2 if form == "int8bal" else 0)
    assert 1 << (bits - 1) <= X < 1 << bits and bits <= 53 * m
    X <<= 53 * m - bits
    return np.array([float(X >> 53 * (m - 1 - t) & (1 << 53) - 1) * 2.0 ** (-53 * (t + 1)) for t in range(m)])


def extreme_pair(rng, S, beta, form, L):
    """Digits of a and b with +-125 modulo 251 at one point for both."""
    p, points = 251, [x for i in range(1, L) for x in (i, 251 - i)]
    while True:
        a = draw_digits(rng, S, beta, form)
        at = [x for x in points if value_at(a, x, beta, form, False, p) in (125, 126)]
        if at:
            break
    while True:
        b = draw_digits(rng, S, beta, form)
        if any(value_at(b, x, beta, form, True, p) in (125, 126) for x in at):
            return a, b


def operands(m, form, S, beta, M, N, K, L):
    """Rows of A and columns of B in turn: a, -a, the largest digits; the
    last of each random."""
    rng = random.Random(m + K)
    a, b = extreme_pair(rng, S, beta, form, L)
    big = largest_digits(S, beta, form)
    out = []
    for digits, n in ((a, M), (b, N)):
        kinds = np.stack([words(digits, m, beta, form), -words(digits, m, beta, form), words(big, m, beta, form)])
        rows = torch.from_numpy(kinds[np.arange(n) % 3].T.copy()).cuda()          # (m, n)
        X = rows[:, :, None].expand(m, n, K).clone()
        gen = np.random.Generator(np.random.PCG64(n))
        X[:, n - 1] = torch.from_numpy(mdinputs.mdouble(gen, m, (K,), ("uniform",))).cuda()
        out.append(X)
    return out[0], out[1].transpose(1, 2).contiguous()


# m, form, S, beta, M, N, K, planes taken
DEEP = [
    (4, "fp64", 10, 21, 256, 256, 65536, True),
    (4, "fp64", 10, 21, 256, 256, 65537, False),
    (8, "int8bal", 52, 8, 128, 128, 65536, True),     # one product of the last diagonal reaches 2^30
    (8, "int8bal", 52, 8, 128, 128, 65537, False),
    (8, "int8", 60, 7, 128, 128, 65536, True),
    (2, "fp64", 5, 21, 300, 200, 2048, True),
    (2, "fp64", 5, 21, 300, 200, 2049, True),
    (8, "int8bal", 52, 8, 130, 100, 2048, True),
    (8, "int8bal", 52, 8, 130, 100, 2049, True),
]


@pytest.mark.parametrize("case", DEEP, ids=lambda c: f"m{c[0]}-{c[1]}-{c[4]}x{c[5]}x{c[6]}")
def test_sums_at_their_bounds(case):
    m, form, S, beta, M, N, K, taken = case
    print(f"[extremes] {case}", flush=True)
    planes = md.lib().md_gemm_planes(md._FORMS[form], M, N, K, S, beta)
    assert (planes > 0) == taken
    A, B = operands(m, form, S, beta, M, N, K, S if form == "fp64" else S // 2)
    C, _ = md.gemm_ex(A, B, form=form, force_S=S, force_beta=beta)
    if taken:
        compare_slices(A, B, C, form, S, beta)
    rows, cols = [0, 1, 2, M - 1], [0, 1, 2, N - 1]
    a, b = A[:, rows].cpu().numpy(), B[:, :, cols].cpu().numpy()
    want = coracle.method_entries(a, b, beta, S, np.arange(4), np.arange(4), balanced=form == "int8bal")[3]
    np.testing.assert_array_equal(C[:, rows][:, :, cols].cpu().numpy(), want)


def compare_slices(A, B, C, form, S, beta):
    M, K, N = A.shape[1], A.shape[2], B.shape[2]
    full, least = md._gemm_sizes(md._FORMS[form], M, N, K, S)
    assert full > 1.4 * least   # the planes do not fit
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    ref, _ = md.gemm_ex(A, B, form=form, force_S=S, force_beta=beta, workspace=ws)
    assert torch.equal(C, ref)


# m, form, S, beta, M, N, K
WIDTHS = [
    (16, "fp64", 45, 20, 129, 140, 200),          # 135 digit bytes: three operands of 64
    (1, "int8bal", 31, 8, 1793, 2050, 2111),
    (2, "int8bal", 31, 8, 1793, 2050, 2111),
    (1, "int8", 30, 7, 1801, 1999, 1985),
    (2, "int8", 30, 7, 1801, 1999, 1985),
]


@pytest.mark.parametrize("case", WIDTHS, ids=lambda c: f"m{c[0]}-{c[1]}-S{c[2]}-{c[4]}x{c[5]}x{c[6]}")
def test_digit_widths(case):
    m, form, S, beta, M, N, K = case
    print(f"[widths] {case}", flush=True)
    assert md.lib().md_gemm_planes(md._FORMS[form], M, N, K, S, beta) > 0
    rng = np.random.Generator(np.random.PCG64(S + m))
    A, B = mdinputs.mdouble(rng, m, (M, K), ("uniform",)), mdinputs.mdouble(rng, m, (K, N), ("log2uniform", 6.0))
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    C, _ = md.gemm_ex(dA, dB, form=form, force_S=S, force_beta=beta)
    compare_slices(dA, dB, C, form, S, beta)
    rows, cols = np.r_[0, 15, 16, M // 2, M - 1], np.r_[0, 17, N // 3, N - 1]
    want = coracle.method_entries(A, B, beta, S, rows, cols, balanced=form == "int8bal")[3]
    np.testing.assert_array_equal(C.cpu().numpy()[:, rows][:, :, cols], want)
