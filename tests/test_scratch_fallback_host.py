"""A product on the library's pool when device memory is short (host only):
the residue contraction and the depth parts are optional, and a call that
does not get their scratch runs the slice products on what those alone take.

The library runs against a stand-in for the HIP runtime's allocation and
launch functions, loaded before it (launches do nothing; device pointers are
numbers): allocations above a size, or beyond a sum, fail.
"""
import json
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
static std::map<uintptr_t, size_t> held;
static uintptr_t next_ptr = 1ull << 40;
static size_t sum, peak, max_one = ~0ull, max_sum = ~0ull;
static int launches, refused;
static uintptr_t last_freed;
static int out_of_order;
extern "C" {
void limits(size_t one, size_t all) { max_one = one; max_sum = all; peak = sum; launches = refused = 0; }
size_t held_now() { return sum; }
size_t held_most() { return peak; }
int launched() { return launches; }
int refusals() { return refused; }
int backwards() { return out_of_order; }
int hipMallocFromPoolAsync(void** p, size_t n, void*, void*)
{
    if (n > max_one || sum + n > max_sum) { ++refused; return 2; }
    *p = (void*)next_ptr;
    held[next_ptr] = n;
    next_ptr += (n + 4095) / 4096 * 4096;
    sum += n;
    peak = sum > peak ? sum : peak;
    return 0;
}
int hipFreeAsync(void* p, void*)
{
    auto it = held.find((uintptr_t)p);
    if (it == held.end()) abort();
    out_of_order += (uintptr_t)p < last_freed;
    last_freed = (uintptr_t)p;
    sum -= it->second;
    held.erase(it);
    return 0;
}
int hipMemPoolCreate(void** pool, const void*) { *pool = malloc(8); return 0; }
int hipMemPoolSetAttribute(void*, int, void*) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return 0; }
int hipMemcpyAsync(void* dst, const void*, size_t n, int, void*) { memset(dst, 0, n); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
struct Dim { unsigned x, y, z; };
int __hipPushCallConfiguration(Dim, Dim, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* s, void** st)
{
    *g = *b = Dim{1, 1, 1};
    *s = 0;
    *st = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { ++launches; return 0; }
}
"""

DRIVER = r"""
import ctypes, json, sys
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
for f in (rt.held_now, rt.held_most, L.md_gemm_workspace_size):
    f.restype = ctypes.c_size_t
i64, i32, P = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p
rt.limits.argtypes = [ctypes.c_size_t, ctypes.c_size_t]
L.md_gemm_planes.argtypes = [i32, i64, i64, i64, i32, i32]
L.md_gemm_ex.argtypes = [i32, i32, i32, i64, i64, i64, P, i64, i64, P, i64, i64, P, i64, i64, P, P]
class Opts(ctypes.Structure):
    _fields_ = [(n, getattr(ctypes, t)) for n, t in json.loads(sys.argv[3])]
ALL = (1 << 64) - 1
def call(m, M, N, K, **kw):
    o = Opts(**kw)
    return L.md_gemm_ex(m, 0, 0, M, N, K, 1 << 44, K, M * K, 1 << 45, N, K * N, 1 << 46, N, M * N,
                        ctypes.byref(o), None)
exec(sys.argv[4])
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    src, so = d / "runtime.cpp", d / "libruntime.so"
    src.write_text(RUNTIME)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    return str(so)


def opts_fields():
    """md_opts as (name, ctypes type) pairs, from the header."""
    text = open(os.path.join(ROOT, "include", "mdgemm.h")).read()
    body = re.search(r"typedef struct md_opts \{(.*?)\} md_opts;", text, re.S).group(1)
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    out = []
    for decl in body.split(";"):
        decl = decl.strip()
        if decl:
            typ, name = re.match(r"(.*?)(\w+)$", decl, re.S).groups()
            out.append((name, "c_void_p" if "*" in typ else "c_size_t" if "size_t" in typ else "c_int"))
    return json.dumps(out)


def drive(runtime, body):
    lib = os.path.join(ROOT, "paper_2606_20863_amd", "libmdgemm.so")
    res = subprocess.run([sys.executable, "-c", DRIVER, runtime, lib, opts_fields(), body],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res
    return [int(x) for x in res.stdout.split()]


def test_digits_are_not_held_twice(runtime):
    """Octo-doubles, 56 balanced digits: the residue planes fail; two digit
    planes of 56 bytes an entry, and not four, fit."""
    rc, refused, rest, planes = drive(runtime, """
n = 1024
rt.limits(ALL, 2 * 56 * n * n + (8 << 20))
rc = call(8, n, n, n, form=2, force_S=56, force_beta=8)
print(rc, rt.refusals(), rt.held_now(), L.md_gemm_planes(2, n, n, n, 56, 8))
""")
    assert planes > 0 and refused > 0
    assert rc == 0 and rest == 0


def test_every_block_of_the_banded_path_finds_a_place(runtime):
    """Hexa-doubles on a hint, validated: statistics, flags, magnitudes,
    digits and the diagonal sums, after the residue planes failed."""
    rc, refused, rest, planes = drive(runtime, """
M, N, K = 256, 256, 1024
rt.limits(200 << 20, ALL)
rc = call(16, M, N, K, form=2, s_hint=105, cert=1 << 47, validate=1)
print(rc, rt.refusals(), rt.held_now(), L.md_gemm_planes(2, M, N, K, 105, 8))
""")
    assert planes > 0 and refused > 0
    assert rc == 0 and rest == 0


def test_depth_parts_yield_to_the_digits(runtime):
    """Quad-doubles times a block of vectors: the parts' integers are left
    out where the digits take what there is."""
    rc, refused, rest, most = drive(runtime, """
M, N, K = 4096, 24, 4096
rt.limits(ALL, ALL)
rc = call(4, M, N, K, form=2, force_S=27, force_beta=8)
most = rt.held_most()
rt.limits(ALL, most - 4096)
rc |= call(4, M, N, K, form=2, force_S=27, force_beta=8)
print(rc, rt.refusals(), rt.held_now(), most)
""")
    assert most > 27 * 4096 * (4096 + 32) + 2 * 8 * 4 * 4096 * 24   # parts in the first call
    assert refused == 1 and rc == 0 and rest == 0


def test_blocks_are_freed_in_the_order_taken(runtime):
    rc, back = drive(runtime, """
rc = call(4, 100, 90, 80, form=2, force_S=27, force_beta=8)
rc |= call(16, 256, 256, 1024, form=2, s_hint=105, cert=1 << 47, validate=1)
print(rc, rt.backwards())
""")
    assert rc == 0 and back == 0
