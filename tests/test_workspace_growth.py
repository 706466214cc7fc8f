"""The library's own workspace on the CPU: the library runs in a process of its own on a stand-in for the HIP runtime whose
allocations can be refused and whose last error, as the runtime's does, stays until it is asked for."""
import re

from test_launch_routes import STAND_IN, run_on_stand_in

# hipMalloc: memory that nothing reads, refused above a bound
MEMORY = r"""
static size_t allowed = (size_t)-1;
static int last_error;
void allow(size_t n) { allowed = n; }
int hipMalloc(void **p, size_t n)
{ if (n > allowed) { *p = 0; return last_error = 2; }
  *p = malloc(1); return 0; }
int hipFree(void *p) { free(p); return 0; }
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


def on_stand_in(d, body):
    stand_in = re.sub(r"int (hipMalloc|hipFree|hipGetLastError)\(.*\n", "", STAND_IN)
    assert "hipMalloc" not in stand_in
    return run_on_stand_in(d, CALLS + body, stand_in + MEMORY)


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
