"""Host build of the kernels' signed rounding steps (``rn_signed`` on
``to_limbs_signed`` limbs, csrc/renorm.h) against the oracle's ``renorm_rn``:
the integers of test_renorm_host.py, and powers of two of either sign (a
negative one has one sign bit more than its magnitude says), all ones and
single bits across the limbs, with units around the subnormal threshold.
"""
import ctypes
import os
import random
import subprocess
from fractions import Fraction

import pytest

from oracle import exact as ox
from test_renorm_host import CSRC, DRIVER, LAYOUTS, cases, columns_of, same_words, value_of


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("renorm_signed")
    src = d / "driver.cpp"
    body = DRIVER.replace("double sgn = to_limbs<T::kCW>(x, L) ? -1.0 : 1.0;",
                          "int32_t sg = to_limbs_signed<T::kCW>(x, L);").replace(
                              "rn_next(L, sgn, scale)", "rn_signed(L, sg, scale)")
    assert "rn_signed" in body and "to_limbs_signed" in body
    src.write_text(body)
    so = d / "librenorm_signed_host.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def powers(nc, cw):
    for e in range(0, cw * (nc - 1) + 60, 7):
        for X in (1 << e, -(1 << e), (1 << e) - 1, -(1 << e) - 1, 3 * (1 << e) >> 1, -((1 << e) + (1 << max(e - 53, 0)))):
            for scale in (0, -e, -1074 - e + 52, -1074 - e + 20, -1075 - e, 900 - e):
                yield columns_of(X, nc, cw), scale, 4


@pytest.mark.parametrize("S,B", LAYOUTS)
def test_signed_steps_match_oracle(lib, S, B):
    nc, cw = lib.layout(S, B, 0), lib.layout(S, B, 2)
    out = (ctypes.c_double * 8)()
    every = list(cases(random.Random(2000 + S), nc, 1500, cw)) + list(powers(nc, cw))
    for cols, scale, m in every:
        lib.renorm(S, B, (ctypes.c_int64 * nc)(*cols), scale, m, out)
        got = list(out)[:m]
        ref = ox.renorm_rn(Fraction(value_of(cols, cw)) * Fraction(2) ** scale, m)
        assert same_words(got, ref), (cols, scale, m, got, ref)
