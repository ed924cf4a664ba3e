"""The work whose speed this library is judged by: m-double matrix products, their training step, batched inner
products and depth-split products, through the package's public entry points, from the launch-bound 64^3 double-double
product to the 4096^3 quad-double one.

A case is a dict of plain values.  ``kind`` is one of

* ``gemm``   one product C = op(A) op(B): ``gemm`` (the default FP64-digit form or an INT8 form), or ``gemm_ex`` with
             transposes or a slice-count hint (``call`` = "hint": what a serving loop does that repeats a shape);
* ``train``  forward and adjoint: ``MDGemm.apply`` and the gradients of both factors for given m-double cotangents;
* ``dot``    a batch of inner products (``dot`` / ``dot_ex``), on the bit pattern of the published experiment;
* ``split``  one product cut along its depth: ``exponents``, a ``gemm_fixed`` per block, ``fixed_add``,
             ``fixed_round``.

Inputs are drawn on the GPU from the seed alone, distributed as ``mdinputs`` draws them (leading words U(-1, 1) or
+-2^U(-r, r), strongly nonoverlapping trailing words; inner products: groups of a leading one and twelve random bits).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2606_20863_amd as md

MAX_COST = 4096.0 ** 3 * 16   # M N K m^2 of the largest listed case (FP64 digits count eightfold)


def listed():
    return [
        # the smallest call: a double-double product whose time is launches and the slice rule's round trip
        {"name": "dd_64", "kind": "gemm", "m": 2, "M": 64, "N": 64, "K": 64, "form": "int8bal", "lead": 0.0,
         "transA": False, "transB": False, "call": "rule"},
        # a matrix against a block of vectors (block Krylov methods, refinement of several right-hand sides)
        {"name": "qd_panel", "kind": "gemm", "m": 4, "M": 4096, "N": 24, "K": 4096, "form": "int8bal", "lead": 0.0,
         "transA": False, "transB": False, "call": "hint"},
        # a ragged quad-double product with a transposed factor, in the published bit fields (sign-magnitude digits)
        {"name": "qd_ragged_int8", "kind": "gemm", "m": 4, "M": 1003, "N": 1517, "K": 1291, "form": "int8", "lead": 4.0,
         "transA": False, "transB": True, "call": "rule"},
        # the medium quad-double workload, wide exponents, repeated with a hint
        {"name": "qd_1024", "kind": "gemm", "m": 4, "M": 1024, "N": 1024, "K": 1024, "form": "int8bal", "lead": 8.0,
         "transA": False, "transB": False, "call": "hint"},
        # the benchmark product: the largest call
        {"name": "qd_4096", "kind": "gemm", "m": 4, "M": 4096, "N": 4096, "K": 4096, "form": "int8bal", "lead": 0.0,
         "transA": False, "transB": False, "call": "rule"},
        # what gemm(A, B) does when no form is named: FP64 digits
        {"name": "qd_default", "kind": "gemm", "m": 4, "M": 1000, "N": 1100, "K": 1200, "form": "fp64", "lead": 0.0,
         "transA": False, "transB": False, "call": "rule"},
        # double-double forward and adjoint, FP64 digits
        {"name": "dd_train_2048", "kind": "train", "m": 2, "M": 2048, "N": 2048, "K": 2048, "form": "fp64", "lead": 0.0},
        # octo-double forward and adjoint, wide exponents
        {"name": "od_train_1024", "kind": "train", "m": 8, "M": 1024, "N": 1024, "K": 1024, "form": "int8bal",
         "lead": 16.0},
        # the widest words
        {"name": "hd_1024", "kind": "gemm", "m": 16, "M": 1024, "N": 1024, "K": 1024, "form": "int8bal", "lead": 6.0,
         "transA": False, "transB": False, "call": "rule"},
        # the published experiment: 1,024 inner products of length 6,144, quad-doubles on a hint, hexa-doubles by rule
        {"name": "qd_dot", "kind": "dot", "m": 4, "batch": 1024, "n": 6144, "form": "int8bal", "call": "hint"},
        {"name": "hd_dot", "kind": "dot", "m": 16, "batch": 1024, "n": 6144, "form": "int8bal", "call": "rule"},
        # a product whose depth is spread over four workers, the exact integers added and rounded once
        {"name": "qd_split", "kind": "split", "m": 4, "M": 2048, "N": 2048, "K": 4096, "form": "int8bal", "blocks": 4},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _slices(form, m):
    """(slice count, digit bits) that a caller fixes for a depth split: the rule's for U(-1, 1) entries."""
    beta, S, _, _ = md.choose_params(form, 4096, 50 * m, 4)
    return S, beta


def draw(rng):
    kind = rng.choice(("gemm", "gemm", "gemm", "train", "dot", "split"))
    form = rng.choice(("int8bal", "int8bal", "int8", "fp64"))
    if kind == "dot":
        m = rng.choice((1, 2, 4, 8, 16))
        batch, n = _size(rng, 1, 4096), _size(rng, 16, 16384)
        while batch * n * m > 1024 * 6144 * 16 or (form == "fp64" and batch * n * m > 1024 * 6144 * 4):
            batch, n = (batch + 1) // 2, (n + 1) // 2
        return {"kind": kind, "m": m, "batch": batch, "n": n, "form": form,
                "call": rng.choice(("rule", "hint")) if form != "fp64" else "rule"}
    m = rng.choice((1, 2, 2, 4, 4, 4, 8, 8, 16))
    M, N, K = (_size(rng, 16, 4096) for _ in range(3))
    cost = (3 if kind == "train" else 1) * m * m * (8 if form == "fp64" else 1)
    while M * N * K * cost > MAX_COST or m * max(M * N, M * K, N * K) > 4 * 4096 ** 2:
        M, N, K = (max(16, (3 * d + 3) // 4) for d in (M, N, K))
    if kind == "split":
        return {"kind": kind, "m": min(m, 8), "M": M, "N": N, "K": max(K, 64), "form": form,
                "blocks": rng.choice((2, 3, 4))}
    case = {"kind": kind, "m": m, "M": M, "N": N, "K": K, "form": form, "lead": rng.choice((0.0, 0.0, 4.0, 8.0))}
    if kind == "gemm":
        case |= {"transA": rng.random() < 0.25, "transB": rng.random() < 0.25,
                 "call": rng.choice(("rule", "hint")) if form != "fp64" else "rule"}
    return case


def _words(gen, m, shape, lead):
    """(m, *shape) m-double entries: leading words U(-1, 1) (lead 0) or +-2^U(-lead, lead), then strongly
    nonoverlapping words w_{t+1} = w_t 2^-53 U(-1, 1), one ulp moved up where that exceeds half an ulp."""
    u = torch.rand(shape, generator=gen, dtype=torch.float64, device="cuda") * 2 - 1
    if lead:
        sign = torch.where(torch.rand(shape, generator=gen, device="cuda") < 0.5, -1.0, 1.0)
        u = torch.exp2(u * lead) * sign
    out = torch.zeros((m,) + tuple(shape), dtype=torch.float64, device="cuda")
    out[0] = u
    inf = torch.full((), math.inf, dtype=torch.float64, device="cuda")
    for t in range(m - 1):
        w = out[t].clone()
        raw = (w * (torch.rand(shape, generator=gen, dtype=torch.float64, device="cuda") * 2 - 1)) * 2.0 ** -53
        ulp = torch.where(w == 0, 0.0, torch.nextafter(w.abs(), inf) - w.abs())
        step = torch.where(raw.abs() > 0.5 * ulp, torch.sign(raw) * ulp, 0.0)
        out[t] = w + step
        out[t + 1] = raw - step
    return out


def _pattern(gen, m, shape):
    """(m, *shape) words of four groups of a leading one and twelve random bits, random signs."""
    out = torch.empty((m,) + tuple(shape), dtype=torch.float64, device="cuda")
    for w in range(m):
        g = torch.randint(0, 1 << 48, shape, generator=gen, dtype=torch.int64, device="cuda")
        mant = torch.zeros_like(g)
        for q in range(4):
            mant = (mant << 13) | (1 << 12) | ((g >> (12 * q)) & 0xfff)
        sign = torch.where(torch.rand(shape, generator=gen, device="cuda") < 0.5, -1.0, 1.0)
        out[w] = sign * (mant.double() * 2.0 ** (-51 - 52 * w))
    return out


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    m = case["m"]
    if case["kind"] == "dot":
        shape = (case["batch"], case["n"])
        return _pattern(gen, m, shape), _pattern(gen, m, shape)
    M, N, K, lead = case["M"], case["N"], case["K"], case.get("lead", 0.0)
    A = _words(gen, m, (K, M) if case.get("transA") else (M, K), lead)
    B = _words(gen, m, (N, K) if case.get("transB") else (K, N), lead)
    if case["kind"] == "train":
        return A, B, _words(gen, m, (M, N), 0.0)
    return A, B


def prepare(case, seed):
    ops = _inputs(case, seed)
    state = {"case": case, "ops": ops}
    if case["kind"] == "train":
        ops[0].requires_grad_(True)
        ops[1].requires_grad_(True)
    elif case["kind"] == "split":
        K, blocks = case["K"], case["blocks"]
        S, beta = _slices(case["form"], case["m"])
        cuts = [K * b // blocks for b in range(blocks + 1)]
        state |= {"S": S, "beta": beta, "nlimb": md.fixed_limbs(beta, S, K),
                  "parts": [(ops[0][:, :, lo:hi], ops[1][:, lo:hi]) for lo, hi in zip(cuts, cuts[1:])],
                  "flags": torch.zeros(1, dtype=torch.int32, device="cuda")}
    elif case["call"] == "hint":
        # the slice count that an earlier call of this shape and kind of data took
        entry = md.dot_ex if case["kind"] == "dot" else md.gemm_ex
        state |= {"hint": entry(*ops, form=case["form"], **_trans(case))[1]["S"], "cert": md.new_cert()}
    return state


def _trans(case):
    return {"transA": case["transA"], "transB": case["transB"]} if case["kind"] == "gemm" else {}


def run(state):
    case, ops = state["case"], state["ops"]
    form = case["form"]
    if case["kind"] == "train":
        A, B, W = ops
        C = md.MDGemm.apply(A, B, form)
        dA, dB = torch.autograd.grad(C, (A, B), W)
        return {"C": C, "dA": dA, "dB": dB}
    if case["kind"] == "split":
        S, beta, nlimb = state["S"], state["beta"], state["nlimb"]
        E, F = md.exponents(*ops)
        total, scale = None, None
        for a, b in state["parts"]:
            X, scale, _ = md.gemm_fixed(a, b, E, F, S=S, beta=beta, form=form, nlimb=nlimb, flags=state["flags"])
            total = X if total is None else md.fixed_add(total, X)
        return {"C": md.fixed_round(total, scale, case["m"]), "X": total, "scale": scale, "flags": state["flags"]}
    if case["call"] == "hint":
        entry = md.dot_ex if case["kind"] == "dot" else md.gemm_ex
        out, _ = entry(*ops, form=form, s_hint=state["hint"], cert=state["cert"], **_trans(case))
        return {"C": out, "cert": state["cert"]}
    if case["kind"] == "dot":
        return {"C": md.dot(*ops, form=form)}
    if case["transA"] or case["transB"]:
        return {"C": md.gemm_ex(*ops, form=form, **_trans(case))[0]}
    return {"C": md.gemm(*ops, form=form)}


def work(case):
    """Each word of the operands read once, each word of the results written once; the multiply-adds of the product
    itself (2 M N K), whatever the number of digit products behind each."""
    m = case["m"]
    if case["kind"] == "dot":
        b, n = case["batch"], case["n"]
        return {"bytes": 8.0 * m * (2 * b * n + b), "flops": 2.0 * b * n}
    M, N, K = case["M"], case["N"], case["K"]
    if case["kind"] == "train":   # A, B, W in; C, dA, dB out
        return {"bytes": 16.0 * m * (M * K + K * N + M * N), "flops": 6.0 * M * N * K}
    out = 8.0 * m * M * N
    if case["kind"] == "split":   # the integers and their scales are results too
        S, beta = _slices(case["form"], m)
        out += 4.0 * (md.fixed_limbs(beta, S, K) + 1) * M * N
    return {"bytes": 8.0 * m * (M * K + K * N) + out, "flops": 2.0 * M * N * K}


def _integers(planes):
    """Exact integers (numpy objects) of m-double planes and the power of two of their unit."""
    w = planes.cpu().numpy()
    mant, e = np.frexp(w)
    e = np.where(w == 0, 0, e) - 53
    unit = int(e[w != 0].min()) if (w != 0).any() else 0
    total = np.zeros(w.shape[1:], dtype=object)
    for t in range(w.shape[0]):
        q = np.ldexp(mant[t], 53).astype(np.int64).astype(object)
        total = total + q * (1 << (np.where(w[t] == 0, 0, e[t] - unit)).astype(object))
    return total, unit


def _rounded(X, unit, m):
    """m planes of the integers X 2^unit, each word the nearest double of what the words before it leave."""
    out = np.zeros((m,) + X.shape)
    for at, x in np.ndenumerate(X):
        for t in range(m):
            if not x:
                break
            shift = max(0, abs(x).bit_length() - 900)   # words past the 900th bit are not reached
            w = float(x >> shift if shift else x)
            x -= int(w) << shift
            out[(t,) + at] = math.ldexp(w, unit + shift)
    return torch.from_numpy(out)


def _product(A, B, m):
    """op(A) op(B): by exact integers where that is quick; else the leading words by FP64 (64 bits hold no more),
    the other words zero."""
    M, K, N = A.shape[1], A.shape[2], B.shape[2]
    if M * N * K <= 3e6 and m * m * (M * K + K * N + M * N) <= 4e6:
        (a, ea), (b, eb) = _integers(A), _integers(B)
        return _rounded(a.dot(b), ea + eb, m)
    out = torch.zeros((m, M, N), dtype=torch.float64, device="cuda")
    out[0] = A.sum(0) @ B.sum(0)
    return out


def exact(case, seed):
    ops, m = _inputs(case, seed), case["m"]
    if case["kind"] == "dot":
        X, Y = ops
        if case["batch"] * case["n"] * m <= 2e6:
            (x, ex), (y, ey) = _integers(X), _integers(Y)
            out = _rounded((x * y).sum(1), ex + ey, m)
        else:
            out = torch.zeros((m, case["batch"]), dtype=torch.float64, device="cuda")
            out[0] = (X.sum(0) * Y.sum(0)).sum(1)
        return {"C": out}
    if case["kind"] == "train":
        A, B, W = ops
        return {"C": _product(A, B, m), "dA": _product(W, B.transpose(1, 2), m),
                "dB": _product(A.transpose(1, 2), W, m)}
    A = ops[0].transpose(1, 2) if case.get("transA") else ops[0]
    B = ops[1].transpose(1, 2) if case.get("transB") else ops[1]
    return {"C": _product(A, B, m)}
