"""The library's own workspace on the CPU: the library runs in a process of its own on a stand-in for the HIP runtime whose
allocations can be refused and whose last error, as the runtime's does, stays until it is asked for."""
import json
import re
import subprocess

import pytest

from paper_2508_03984_amd import build
from test_launch_routes import STAND_IN, run_on_stand_in

# hipMalloc: memory that nothing reads, refused above a bound
MEMORY = r"""
static size_t allowed = (size_t)-1;
static int last_error, asked, freed;
void allow(size_t n) { allowed = n; }
int times_asked(void) { return asked; }
int times_freed(void) { return freed; }
int hipMalloc(void **p, size_t n)
{ ++asked;
  if (n > allowed) { *p = 0; return last_error = 2; }
  *p = malloc(1); return 0; }
int hipFree(void *p) { freed += p != 0; free(p); return 0; }
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
"""
CALLS = r"""
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.launched.restype = C.c_char_p
fake.allow.argtypes = [C.c_size_t]
lib = C.CDLL(sys.argv[2])
vp, i64, sz = C.c_void_p, C.c_int64, C.c_size_t
lib.oz2_create.argtypes = [C.POINTER(vp)]
lib.oz2_destroy.argtypes = [vp]
lib.oz2_ctx_dgemm.argtypes = [vp, C.c_int, C.c_int, C.c_int, i64, i64, i64, C.c_double, vp, i64, vp, i64, C.c_double, vp, i64, C.c_int, vp]
lib.oz2_prepare_d.argtypes = [C.c_int, C.c_int, i64, i64, vp, i64, C.c_int, vp, C.POINTER(vp)]
lib.oz2_ctx_dgemm_prepared.argtypes = [vp, vp, vp, C.c_double, C.c_double, vp, i64, vp]
lib.oz2_ctx_workspace_bytes.argtypes = [vp, i64, i64, i64, C.c_int]
lib.oz2_ctx_workspace_bytes.restype = sz
lib.oz2_ctx_set_workspace_limit.argtypes = [vp, sz]
lib.oz2_operand_free.argtypes = [vp]
X = 1 << 20                                               # nothing reads it

def context():
    c = vp()
    assert lib.oz2_create(C.byref(c)) == 0
    return c

def call(c, m, n, k, N, allow=2**63):
    fake.forget()
    fake.allow(allow)
    status = lib.oz2_ctx_dgemm(c, 0, 0, 0, m, n, k, 1.0, X, k, X, n, 0.0, X, n, N, None)
    return status, fake.launched().decode().split("\n")[:-1]

def prepared(c, m, n, k, N, allow=2**63):
    fake.allow(2**63)
    a, b = vp(), vp()
    assert lib.oz2_prepare_d(0, 0, m, k, X, k, N, None, C.byref(a)) == 0
    assert lib.oz2_prepare_d(1, 0, n, k, X, n, N, None, C.byref(b)) == 0
    fake.forget()
    fake.allow(allow)                                     # for the product: the operands have buffers of their own
    status = lib.oz2_ctx_dgemm_prepared(c, a, b, 1.0, 0.0, X, n, None)
    names = fake.launched().decode().split("\n")[:-1]
    lib.oz2_operand_free(a); lib.oz2_operand_free(b)
    return status, names

"""


def on_stand_in(d, body, data=None):
    stand_in = re.sub(r"int (hipMalloc|hipFree|hipGetLastError)\(.*\n", "", STAND_IN)
    assert "hipMalloc" not in stand_in
    return run_on_stand_in(d, CALLS + body, stand_in + MEMORY, data=json.dumps(data))


def in_ranges(names):
    return any("k_epilogue_ranges" in n for n in names)


def test_call_without_room_for_the_planes_of_k_ranges(tmp_path):
    """Where the buffer with the planes of the K ranges is not to be had and the one without them is, the call runs, with one range."""
    got = on_stand_in(tmp_path, r"""
out = []
m, n, k, N = 256, 256, 40000, 16
for product in (call, prepared):
    c = context()
    whole = product(c, m, n, k, N)                        # everything to be had
    lib.oz2_destroy(c)
    c = context()
    one_range = N * 65536 + (lib.oz2_ctx_workspace_bytes(c, m, n, k, N) - 4 * N * 65536 if product is call else 0)
    tight = product(c, m, n, k, N, allow=one_range)
    out.append([whole, tight, call(c, 64, 64, 64, 2)])
    lib.oz2_destroy(c)
print(json.dumps(out))
""")
    assert len(got) == 2
    for whole, tight, again in got:
        assert whole[0] == 0 and in_ranges(whole[1])
        assert tight[0] == 0 and again[0] == 0, (tight, again)
        assert not in_ranges(tight[1]) and "k_epilogue" in tight[1][-1]
        assert len(tight[1]) == len(whole[1])


def test_refused_altogether(tmp_path):
    """No buffer at all: a status, nothing launched, and the next call runs."""
    got = on_stand_in(tmp_path, r"""
c = context()
refused = call(c, 256, 256, 40000, 16, allow=4096)
print(json.dumps([refused, call(c, 256, 256, 40000, 16)]))
""")
    assert got[0] == [3, []]
    assert got[1][0] == 0 and in_ranges(got[1][1])


# (product, m, n, k, N) one after another on one context, and whether the last one runs in K ranges
ORDERS = {
    "prepared, the same C with a short k first": ([("prepared", 256, 256, 2048, 16), ("prepared", 256, 256, 40000, 16)], True),
    "prepared, 512": ([("prepared", 512, 512, 1000, 16), ("prepared", 512, 512, 40000, 16)], True),
    "prepared, 768": ([("prepared", 768, 768, 1000, 16), ("prepared", 768, 768, 40000, 16)], True),
    "prepared, one tile": ([("prepared", 100, 100, 600, 2), ("prepared", 100, 100, 131072, 2)], True),
    "a buffer between the two sizes": ([("call", 2048, 1536, 4864, 16), ("call", 256, 256, 40000, 16)], True),
    "a large one first": ([("call", 4096, 4096, 4096, 14), ("call", 1280, 1024, 40000, 16)], True),
    "prepared after a call": ([("call", 300, 300, 300, 14), ("prepared", 256, 256, 40000, 16)], True),
    "no ranges to be had": ([("prepared", 256, 256, 40000, 16), ("prepared", 256, 256, 1000, 16)], False),
}


@pytest.fixture(scope="module")
def orders(tmp_path_factory):
    return on_stand_in(tmp_path_factory.mktemp("orders"), r"""
products = {"call": call, "prepared": prepared}
out = {}
for name, calls in json.loads(sys.stdin.read()).items():
    c = context()
    for product, *sizes in calls:
        last = products[product](c, *sizes)
    freed = fake.times_freed()
    again = products[product](c, *sizes)
    out[name] = [last, again, fake.times_freed() - freed - (2 if product == "prepared" else 0)]
    lib.oz2_destroy(c)
print(json.dumps(out))
""", data={name: calls for name, (calls, _) in ORDERS.items()})


@pytest.mark.parametrize("name", sorted(ORDERS))
def test_k_ranges_whatever_came_first(orders, name):
    """What a product launches does not depend on the calls before it, and a call that has run keeps its buffer."""
    last, again, freed = orders[name]
    assert last[0] == 0 and again == last
    assert in_ranges(last[1]) == ORDERS[name][1], last
    assert freed == 0


def test_planes_never_make_the_buffer_grow(tmp_path):
    """A graph may hold the buffer that a call has run in: a product that lacks nothing but planes leaves it where it is, also where
    the reserve was refused, or limited."""
    got = on_stand_in(tmp_path, r"""
out = []
short, long_ = (256, 256, 2048, 16), (256, 256, 40000, 16)
for limit, allowed in ((0, 2**63), (0, 65536 * 16), (65536 * 16, 2**63), (65536 * 16 * 4, 2**63)):
    c = context()
    lib.oz2_ctx_set_workspace_limit(c, limit)
    a = [prepared(c, *short, allow=allowed)]
    asked, freed = fake.times_asked(), fake.times_freed()
    a.append(prepared(c, *long_, allow=allowed))
    out.append(a + [fake.times_asked() - asked - 2, fake.times_freed() - freed - 2])    # but for the operands
    lib.oz2_destroy(c)
print(json.dumps(out))
""")
    for (short, long_, asked, freed), ranges in zip(got, (True, False, False, True)):
        assert short[0] == long_[0] == 0 and asked == freed == 0
        assert not in_ranges(short[1]) and in_ranges(long_[1]) == ranges


RESERVE = r"""
#include <cstdio>
#include "oz2_plan.hpp"
using namespace oz2;
int main() {
    long bad = 0, products = 0;
    size_t most = 0;
    for (int hm = 1; hm <= 896; ++hm)                         // blocks of 128 rows and columns: up to 448 tiles of 256
        for (int hn = 1; hn <= 896 && ((hm + 1) / 2) * ((hn + 1) / 2) <= 224; ++hn)
            for (int N = 2; N <= 20 && ((hm + 1) / 2) * ((hn + 1) / 2) * N <= 448; ++N)
                for (int inside : {1, 128})                   // of the last block
                    for (int64_t k = 1536; k <= OZ2_MAX_K; k += 128) {
                        const Layout L = make_layout(128 * (hm - 1) + inside, 128 * (hn - 1) + inside, k, N, true, false);
                        ++products;
                        most = std::max(most, L.prod_ranges);
                        if (L.prod_ranges > planes_reserve(L.prod_whole)) ++bad;
                    }
    std::printf("bad=%ld %d %d\n", bad, products > 1000000, most > kMaxPlanes / 2);
    return bad != 0;
}
"""


def test_the_reserve_covers_every_plan(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(RESERVE)
    exe = tmp_path / "main"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "bad=0 1 1", out.stdout
