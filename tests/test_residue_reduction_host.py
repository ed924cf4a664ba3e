"""The residues' reduction modulo a prime (``residue_f32`` and
``residue_wide``, csrc/resid.hip) compiled for the host, for all eight primes:
every value that the evaluation can hand to the one-step form, every sum of
products that 2,048 depths can give it, and for the two-step form sums up to
65,536 depths, at both ends, around the middle between multiples of p (where a
quotient off by one would show) and spread over the rest.  A result has to be
congruent, to fit a byte, and from the evaluation to be centred (the sums'
bound is 65,536 (p - 1)^2 / 4 < 2^31).
"""
import ctypes
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_20863_amd", "csrc")
PRIMES = (251, 241, 239, 233, 229, 227, 223, 211)

DRIVER = r"""
#include <cstdint>
#include <cstdlib>
#define __device__
#define __forceinline__ inline
static inline int __mul24(int a, int b)
{
    const int64_t x = (int64_t)(int32_t)((uint32_t)a << 8) >> 8, y = (int64_t)(int32_t)((uint32_t)b << 8) >> 8;
    return (int)(uint32_t)(uint64_t)(x * y);
}
FUNCTIONS
// The largest |r| over v = lo, lo + step, .. <= hi, -1 where one is wrong;
// r is the low byte, as it is stored.
template <class F>
static int scan(F f, int64_t lo, int64_t hi, int64_t step, int p)
{
    int most = 0;
    for (int64_t v = lo; v <= hi; v += step) {
        const int r = (int8_t)f((int)v);
        if ((v - r) % p)
            return -1;
        most = abs(r) > most ? abs(r) : most;
    }
    return most;
}
extern "C" {
int one_step(int p, int64_t lo, int64_t hi, int64_t step)
{
    return scan([=](int v) { return residue_f32(v, 1.0f / (float)p, -p); }, lo, hi, step, p);
}
int two_steps(int p, int64_t lo, int64_t hi, int64_t step)
{
    return scan([=](int v) { return residue_wide(v, 1.0f / (float)p, -p); }, lo, hi, step, p);
}
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("residue")
    text = open(os.path.join(CSRC, "resid.hip")).read()
    found = [re.search(rf"__device__ __forceinline__ int {n}\(.*?\n}}\n", text, re.S).group(0)
             for n in ("residue_f32", "residue_wide")]
    (d / "driver.cpp").write_text(DRIVER.replace("FUNCTIONS", "\n".join(found)))
    so = d / "libresidue.so"
    subprocess.run(["g++", "-std=c++20", "-O2", "-mfma", "-ffp-contract=off", "-shared", "-fPIC",
                    str(d / "driver.cpp"), "-o", str(so)], check=True)
    L = ctypes.CDLL(str(so))
    for f in (L.one_step, L.two_steps):
        f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3
    return L


@pytest.mark.parametrize("p", PRIMES + (256,))
def test_evaluation_is_centred(lib, p):
    """|v| < 2^22 covers 192 digit bytes times weights of at most 127; modulus
    256 (the last diagonal's rows) takes one digit as it is."""
    if p == 256:
        assert lib.one_step(p, -128, 127, 1) == 128
    else:
        assert lib.one_step(p, -(1 << 22) + 1, (1 << 22) - 1, 1) == (p - 1) // 2


@pytest.mark.parametrize("p", PRIMES)
def test_one_step_up_to_2048_depths(lib, p):
    most = 2048 * ((p - 1) // 2) ** 2
    assert 0 <= lib.one_step(p, -most, most, 1) <= 127


@pytest.mark.parametrize("p", PRIMES)
def test_two_steps_up_to_65536_depths(lib, p):
    most = 65536 * ((p - 1) // 2) ** 2
    assert most < 1 << 30
    middle, first = (p - 1) // 2, -(most // p) * p
    for lo in (-most, -1000000, most - 2000000):
        assert lib.two_steps(p, lo, lo + 2000000, 1) == middle
    for lo, step in ((first + middle, 17 * p), (first + middle + 1, 17 * p), (-most, 1009)):
        assert 0 <= lib.two_steps(p, lo, most, step) <= middle
