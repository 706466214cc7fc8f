"""Which kernels a call launches, seen on the CPU: the library runs in a process of its own on a stand-in for the HIP
runtime that records the launches and does nothing else."""
import json
import os
import re
import subprocess
import sys

import pytest

STAND_IN = r"""
#include <stddef.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void *host; const char *name; } known[4096];
static int n_known;
static char names[1 << 20];
static dim3 g_, b_; static size_t s_; static void *st_;
static void *module;
void **__hipRegisterFatBinary(const void *d) { (void)d; return &module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g)
{ (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned l, void *t, void *b, void *bd,
                           void *gd, int *w)
{ (void)m; (void)dev; (void)l; (void)t; (void)b; (void)bd; (void)gd; (void)w;
  if (n_known < 4096) { known[n_known].host = host; known[n_known++].name = strdup(name); } }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *st) { g_ = g; b_ = b; s_ = s; st_ = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st) { *g = g_; *b = b_; *s = s_; *st = st_; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t s, void *st)
{ (void)g; (void)b; (void)a; (void)s; (void)st;
  for (int i = 0; i < n_known; ++i)
      if (known[i].host == f && strlen(names) + strlen(known[i].name) + 2 < sizeof names)
      { strcat(names, known[i].name); strcat(names, "\n"); break; }
  return 0; }
const char *launched(void) { return names; }
void forget(void) { names[0] = 0; }
int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { (void)p; (void)d; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)p; (void)s; return 1; }
int hipDeviceSynchronize(void) { return 0; }
int hipEventCreate(void **e) { *e = &module; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = &module; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 0; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = &module; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
"""

CALLER = r"""
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)            # its name is the runtime's: the library binds to it
fake.launched.restype = C.c_char_p
lib = C.CDLL(sys.argv[2])
vp, i64 = C.c_void_p, C.c_int64
for t in "ds":
    f = getattr(lib, "oz2_prepare_" + t)
    f.argtypes = [C.c_int, C.c_int, i64, i64, vp, i64, C.c_int, vp, C.POINTER(vp)]
lib.oz2_operand_free.argtypes = [vp]
out = {}
for option in (1, 0):
    lib.oz2_set_small_conversion(option)
    for t in "ds":
        for side, op, rows, k in ((0, 0, 40, 300), (1, 0, 40, 300), (0, 1, 33, 4096), (1, 1, 10, 16384),
                                  (1, 0, 10, 4097), (0, 0, 10, 16385)):
            fake.forget()
            h = vp()
            X = 1 << 20                                   # nothing reads it
            status = getattr(lib, "oz2_prepare_" + t)(side, op, rows, k, X, max(rows, k), 3, None, C.byref(h))
            assert status == 0, status
            out["%d %s %d %d %d" % (option, t, side, op, k)] = fake.launched().decode().split("\n")[:-1]
            lib.oz2_operand_free(h)
print(json.dumps(out))
"""


def run_on_stand_in(d, caller, stand_in=STAND_IN, data=None):
    """What `caller` prints (JSON) about a library whose HIP runtime is the stand-in, in a process of its own."""
    import paper_2508_03984_amd as oz
    if not os.path.exists(oz.lib_path()):
        from paper_2508_03984_amd.build import build_library
        build_library()
    needed = subprocess.run(["readelf", "-d", oz.lib_path()], capture_output=True, text=True, check=True).stdout
    soname = next(line.split("[")[1].split("]")[0] for line in needed.splitlines() if "libamdhip64" in line)
    (d / "fake.c").write_text(stand_in)
    (d / "fake.map").write_text("hip_4.2 { global: *; };\nhip_6.0 { global: hipGetDevicePropertiesR0600; } hip_4.2;\n")
    (d / "caller.py").write_text(caller)
    fake = d / "libfake.so"
    subprocess.check_call(["gcc", "-std=gnu99", "-O1", "-shared", "-fPIC", "-Wl,-soname," + soname,
                           "-Wl,--version-script=" + str(d / "fake.map"), str(d / "fake.c"), "-o", str(fake)])
    run = subprocess.run([sys.executable, str(d / "caller.py"), str(fake), oz.lib_path()], input=data, capture_output=True,
                         text=True)
    assert run.returncode == 0, run.stderr
    return json.loads(run.stdout)


@pytest.fixture(scope="module")
def prepare_launches(tmp_path_factory):
    return run_on_stand_in(tmp_path_factory.mktemp("routes"), CALLER)


def test_prepared_operands_follow_the_conversion_option(prepare_launches):
    """Vectors that fit a workgroup take the fused conversion, and the general kernels if the option is off; longer
    ones take the general kernels anyway."""
    assert len(prepare_launches) == 24
    for case, names in prepare_launches.items():
        option, _, side, op, k = case.split()
        rows = side == op
        fits = int(k) <= (16384 if rows else 4096)
        fused = [n for n in names if "k_convert" in n]
        assert names, case
        if option == "1" and fits:
            assert len(names) == 1 and fused, (case, names)
        else:
            assert not fused and len(names) >= 2, (case, names)


PRODUCTS = r"""
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.launched.restype = C.c_char_p
lib = C.CDLL(sys.argv[2])
vp, i64 = C.c_void_p, C.c_int64
for t, real in (("d", C.c_double), ("s", C.c_float)):
    getattr(lib, "oz2_prepare_" + t).argtypes = [C.c_int, C.c_int, i64, i64, vp, i64, C.c_int, vp, C.POINTER(vp)]
    getattr(lib, "oz2_%sgemm_prepared" % t).argtypes = [vp, vp, real, real, vp, i64, vp]
    getattr(lib, "oz2_%sgemm_op" % t).argtypes = [C.c_int, C.c_int, C.c_int, i64, i64, i64, real, vp, i64, vp, i64, real, vp, i64, C.c_int, vp]
lib.oz2_operand_free.argtypes = [vp]
out = {}
X = 1 << 20                                               # nothing reads it
for case in json.loads(sys.stdin.read()):
    t, m, n, k, N = case
    got = []
    for accurate in (0, 1):
        fake.forget()
        assert getattr(lib, "oz2_%sgemm_op" % t)(0, 0, accurate, m, n, k, 1.0, X, k, X, n, 0.0, X, n, N, None) == 0
        got.append(fake.launched().decode().split("\n")[:-1])
    a, b = vp(), vp()
    assert getattr(lib, "oz2_prepare_" + t)(0, 0, m, k, X, k, N, None, C.byref(a)) == 0
    assert getattr(lib, "oz2_prepare_" + t)(1, 0, n, k, X, n, N, None, C.byref(b)) == 0
    fake.forget()
    assert getattr(lib, "oz2_%sgemm_prepared" % t)(a, b, 1.0, 0.0, X, n, None) == 0
    got.append(fake.launched().decode().split("\n")[:-1])
    lib.oz2_operand_free(a); lib.oz2_operand_free(b)
    out["%s %d %d %d %d" % tuple(case)] = got
print(json.dumps(out))
"""

# A product that converts its factors in two launches (GEMMs, accumulation) or one; prepared operands take one for all of these.
TWO = [("d", 300, 300, 128, 15), ("d", 400, 400, 256, 15), ("s", 400, 400, 384, 8), ("d", 448, 448, 256, 16), ("d", 200, 200, 256, 16),
       ("d", 65, 66, 100, 16), ("d", 384, 384, 128, 17), ("d", 512, 512, 128, 16), ("d", 512, 130, 128, 16), ("s", 300, 300, 257, 7)]
ONE = [("d", 256, 256, 256, 14), ("d", 256, 256, 256, 15), ("d", 64, 64, 64, 20), ("d", 512, 128, 128, 16), ("d", 100, 401, 256, 16),
       ("d", 449, 449, 256, 16), ("d", 385, 385, 128, 17), ("s", 400, 400, 256, 8), ("s", 400, 400, 256, 10), ("s", 300, 300, 512, 6),
       ("s", 449, 300, 500, 8), ("d", 449, 512, 128, 13), ("d", 64, 250, 256, 16),
       ("d", 8000, 30, 64, 15), ("d", 1, 1, 1, 2)]

# Products whose INT8 GEMM has 127 to 129 tiles of 256 x 256 or thereabouts, and 256 and 272 of 128 x 128
TILES = [("s", 1024, 1024, 600, 8), ("d", 2048, 2048, 600, 2), ("d", 256, 256 * 43, 600, 3), ("d", 512, 512, 600, 16),
         ("d", 512, 512, 600, 17), ("s", 1024, 1024, 600, 9), ("d", 2048, 4096, 600, 14), ("d", 2304, 4096, 600, 14)]


@pytest.fixture(scope="module")
def product_launches(tmp_path_factory):
    return run_on_stand_in(tmp_path_factory.mktemp("products"), PRODUCTS, data=json.dumps(TWO + ONE + [("d", 100, 100, 513, 7)] + TILES))


def test_one_launch_form_where_it_gains(product_launches):
    """The one-launch form of the smallest products is taken by calls that convert their factors only where it is the
    faster one, by prepared operands throughout."""
    for case in TWO + ONE:
        fast, accurate, prepared = product_launches["%s %d %d %d %d" % case]
        one = case in ONE
        assert ("k_tiny_product" in " ".join(fast)) == one and ("k_epilogue" in " ".join(fast)) != one, case
        assert ("k_tiny_product" in " ".join(accurate)) == one and ("k_epilogue" in " ".join(accurate)) != one, case
        assert len(prepared) == 1 and "k_tiny_product" in prepared[0], case
        assert len(fast) == (2 if one else 3), (case, fast)
    for names in product_launches["d 100 100 513 7"]:     # beyond the limits of the form
        assert "k_tiny_product" not in " ".join(names) and "k_epilogue" in names[-1]


def test_tiles_of_the_gemm(product_launches):
    """Tiles of 128 x 128 up to 128 tiles of 256 x 256, 8 wavefronts while each has a compute unit; accurate mode's one slice by the
    same rule."""
    def tile(names):
        return [re.search(r"k_int8_gemm(?:_persistent)?I((?:Li\d+E){6})", n).group(1) for n in names if "k_int8_gemm" in n]

    def blocks(n):
        return (n + 255) // 256

    def expected(large):
        return ("Li2ELi4ELi2ELi1ELi64ELi6E" if 4 * large <= 256 else "Li2ELi2ELi2ELi2ELi64ELi4E") if large <= 128 else "Li2ELi4ELi4ELi2ELi64ELi4E"
    seen = set()
    for case in TILES:
        fast, accurate, prepared = product_launches["%s %d %d %d %d" % case]
        slice_ = blocks(case[1]) * blocks(case[2])
        assert tile(fast) == tile(prepared) == [expected(slice_ * case[4])], case
        assert tile(accurate) == [expected(slice_), expected(slice_ * case[4])], case
        seen |= {slice_, slice_ * case[4]}
    assert {64, 68, 128, 129, 144} <= seen
