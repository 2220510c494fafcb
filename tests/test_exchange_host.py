"""Host side of bls_embbag_pool_exchange without a GPU: a few HIP runtime calls are replaced by a library that notes them and
fails one launch on request.  No kernel runs; the calls' order and what they leave of the ring are what is looked at."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
char noted[4096];                       /* L launch, W wait, R record; the stream's digit behind each */
int launches_left = -1, waits_left = -1;   /* that many succeed, the next one fails; -1: all succeed */
unsigned grid_y;                        /* of the latest launch */
static int last;
static int len;
static void note(char c, size_t s) { noted[len++] = c; noted[len++] = (char)('0' + s % 10); noted[len] = 0; }
void forget(void) { len = 0; noted[0] = 0; }
typedef struct { unsigned x, y, z; } dim3;
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { return 0; }
int hipStreamSynchronize(void *st) { return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { *e = (void *)16; return 0; }
int hipEventDestroy(void *e) { return 0; }
int hipEventRecord(void *e, void *st) { note('R', (size_t)st); return 0; }
int hipStreamWaitEvent(void *st, void *e, unsigned f) { if (waits_left == 0) return 1; if (waits_left > 0) --waits_left; note('W', (size_t)st); return 0; }
static dim3 grid, block;                /* what <<< >>> hands to the launch that follows */
static size_t lds;
static void *queue;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, void *st) { grid = g; block = b; lds = sh; queue = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, void **st) { *g = grid; *b = block; *sh = lds; *st = queue; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t sh, void *st)
{
    if (launches_left == 0) return last = 1;
    if (g.x == 0 || g.y == 0 || g.z == 0) return last = 9;   /* as the runtime: invalid configuration */
    if (launches_left > 0) --launches_left;
    grid_y = g.y;
    note('L', (size_t)st);
    return 0;
}
int hipGetLastError(void) { int e = last; last = 0; return e; }
"""

DRIVER = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
noted = C.c_char.in_dll(stub, "noted")
left, waits = C.c_int.in_dll(stub, "launches_left"), C.c_int.in_dll(stub, "waits_left")
class Config(C.Structure):
    _fields_ = [("P", C.c_int32), ("T", C.c_int32), ("D", C.c_int32), ("k", C.c_int32), ("B", C.c_int64), ("table_dtype", C.c_int32),
                ("part_kind", C.c_int32), ("rows", C.POINTER(C.c_int64)), ("table_owner", C.POINTER(C.c_int32))]
vp = C.c_void_p
at = lambda n: vp(0x10000 * n)                                # 16-byte aligned, never followed
def ctx(k, D=64, dtype=0, B=64, part=0, T=2):
    h = vp()
    rows, own = (C.c_int64 * T)(*[9] * T), (C.c_int32 * T)(*[t % 2 for t in range(T)])
    assert L.bls_create(C.byref(Config(2, T, D, k, B, dtype, part, rows, own)), C.byref(h)) == 0
    for t in range(T):
        for rank, n in ((t % 2, 9),) if part == 0 else ((0, 5), (1, 4)):
            assert L.bls_set_shard(h, t, rank, at(1), C.c_int64(n)) == 0
    n = C.c_size_t()
    assert L.bls_desc_bytes(h, C.byref(n)) == 0
    assert L.bls_commit(h, at(2), n, None) == 0
    assert L.bls_set_ring(h, at(3), C.c_size_t(1 << 40)) == 0
    return h
def ring(h):
    a, b, k = C.c_int64(), C.c_int64(), C.c_int32()
    assert L.bls_ring_state(h, C.byref(a), C.byref(b), C.byref(k)) == 0
    return a.value, b.value
L.bls_last_error.restype = C.c_char_p
def issue(h, st, nnz=100):
    stub.forget()
    it, slot = C.c_int64(-1), C.c_int32(-1)
    rc = L.bls_embbag_pool_exchange(h, at(4), at(5), C.c_int64(nnz), at(6), at(7), C.byref(it), C.byref(slot), vp(st))
    return rc, it.value, slot.value, C.string_at(C.addressof(noted)).decode()
def unpack(h, it, st):
    stub.forget()
    rc = L.bls_unpack(h, C.c_int64(it), at(8), vp(st))
    return rc, C.string_at(C.addressof(noted)).decode()
"""


def run(tmp_path, body):
    import paper_2512_19342_amd as pkg
    if not os.path.exists(pkg.lib_path()):
        from paper_2512_19342_amd import build
        build.build()
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    src, so, py = tmp_path / "runtime.c", tmp_path / "runtime.so", tmp_path / "driver.py"
    src.write_text(RUNTIME)
    py.write_text(DRIVER + body)
    subprocess.check_call([cc, "-shared", "-fPIC", "-O1", str(src), "-o", str(so)])
    r = subprocess.run([sys.executable, str(py), str(so), pkg.lib_path()], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout


def test_a_failed_launch_leaves_the_ring_alone(tmp_path):
    run(tmp_path, r"""
for k in (1, 3):
    h = ctx(k)
    assert issue(h, 0) == (0, 0, 0, "L0R0")                   # one launch, the slot's event
    assert unpack(h, 0, 0) == (0, "L0R0")
    left.value = 0
    rc, it, slot, calls = issue(h, 0)
    assert rc != 0 and calls == "" and (it, slot) == (-1, -1) and ring(h) == (1, 1), (rc, it, slot, calls, ring(h))
    left.value = -1
    assert issue(h, 0) == (0, 1, 1 % k, "L0R0") and ring(h) == (2, 1)
    assert unpack(h, 1, 0)[0] == 0 and ring(h) == (2, 2)
""")


def test_the_slot_is_waited_for_only_before_it_is_written(tmp_path):
    """Another stream's copy-out may be late: what does not touch the slot runs before the wait.  Stream order alone needs
    neither a wait nor a second launch."""
    run(tmp_path, r"""
for k in (1, 2):
    h = ctx(k)
    for it in range(6):                                       # issued on stream 1, copied out by stream 2
        rc, j, slot, calls = issue(h, 1)
        assert (rc, j, slot) == (0, it, it % k)
        assert calls == ("L1R1" if it < k else "L1W1L1R1"), (k, it, calls)
        assert unpack(h, it, 2) == (0, "W2L2R2")
    h = ctx(k)
    for it in range(4):
        assert issue(h, 3)[3] == "L3R3" and unpack(h, it, 3) == (0, "L3R3")
    # the wait fails: the ring is as it was
    h = ctx(1)
    assert issue(h, 1)[0] == 0 and unpack(h, 0, 2)[0] == 0
    waits.value = 0
    rc, j, slot, calls = issue(h, 1)
    waits.value = -1
    assert rc != 0 and (j, slot) == (-1, -1) and ring(h) == (1, 1) and issue(h, 1)[3] == "L1W1L1R1"
    # the second launch fails: the iteration has been started, as the separate calls leave it
    h = ctx(1)
    assert issue(h, 1)[0] == 0 and unpack(h, 0, 2)[0] == 0
    left.value = 1
    rc, j, slot, calls = issue(h, 1)
    left.value = -1
    assert rc != 0 and (j, slot) == (1, 0) and calls == "L1W1" and ring(h) == (2, 1)
    assert L.bls_alltoallv_local(h, at(7), C.c_int32(0), vp(1)) == 0 and unpack(h, 1, 1)[0] == 0
""")


def test_one_launch_only_where_its_stores_are_worth_it(tmp_path):
    """Two tables, by storage, partition, length, megabytes of vectors and rows a segment: either side of every line; the
    other sizes take the separate calls (pool, pack, exchange)."""
    run(tmp_path, r"""
fp32, fp16, u8, f8 = 0, 1, 2, 3
one, apart = "L0R0", "L0L0L0R0"
for dtype, mb, rows, calls in ((u8, 24, 1, one), (f8, 25, 1, apart), (u8, 24, 12, one), (f8, 24, 13, apart), (u8, 16, 99, one),
                               (u8, 17, 99, apart), (fp16, 24, 99, one), (fp16, 25, 32, one), (fp16, 25, 33, apart),
                               (fp32, 25, 99, one), (fp32, 999, 0, one), (u8, 24, 0, one), (u8, 25, 0, apart)):
    B = (mb << 20) // (2 * 64 * 4)
    h = ctx(1, dtype=dtype, B=B)
    got = issue(h, 0, int(2 * B * rows))
    assert got == (0, 0, 0, calls), (dtype, mb, rows, got)
    assert unpack(h, 0, 0)[0] == 0 and ring(h) == (1, 1)
for dtype, part, D, mb, calls in ((fp32, 0, 20, 48, one), (fp32, 0, 20, 49, apart), (fp32, 0, 60, 49, apart), (fp32, 0, 64, 49, one), (fp32, 0, 68, 999, one),
                                  (fp32, 0, 48, 999, one), (fp32, 1, 28, 96, one), (fp32, 1, 28, 97, apart), (fp32, 1, 36, 999, one),
                                  (fp16, 0, 40, 49, apart), (fp16, 0, 72, 999, one), (fp16, 1, 24, 97, apart), (fp32, 0, 33, 999, one)):
    B = (mb << 20) // ((1 + part) * 2 * D * 4)
    h = ctx(1, D=D, dtype=dtype, B=B, part=part)
    got = issue(h, 0, 2 * B)
    assert got == (0, 0, 0, calls), (dtype, part, D, mb, got)
for rows, calls in ((4, one), (5, apart)):
    h = ctx(1, D=28)
    assert issue(h, 0, 2 * 64 * rows) == (0, 0, 0, calls)
""")


def test_few_shards_are_spread_over_the_whole_chip(tmp_path):
    """Three stores of shards that would keep under seven tenths of the eight XCDs busy: a grid with a row per shard in place of
    the flat one that deals shards to XCDs, unless bls_set_pool_tuning asks for the deal."""
    run(tmp_path, r"""
grid_y = C.c_uint.in_dll(stub, "grid_y")
for T, y in ((1, 1), (2, 2), (5, 5), (6, 1), (8, 1), (9, 9), (11, 11), (12, 1), (16, 1), (17, 1)):
    h = ctx(1, T=T)
    assert issue(h, 0)[0] == 0 and grid_y.value == y, (T, grid_y.value)
    assert L.bls_set_pool_tuning(h, 0, 0, 1, -1) == 0 and unpack(h, 0, 0)[0] == 0
    assert issue(h, 0)[0] == 0 and grid_y.value == 1, T
""")


def test_a_rank_without_tables_takes_part(tmp_path):
    """One table, owned by rank 0: rank 1 has nothing to pool, and its put is its arrival alone."""
    run(tmp_path, r"""
h = ctx(1, T=1)
for it in range(3):
    for rank in range(2):
        stub.forget()
        assert L.bls_rank_put(h, rank, at(4), None, at(5), C.c_int64(100), C.c_int64(it), vp(rank + 1)) == 0, (it, rank)
        waits_first = "" if it == 0 else f"W{rank + 1}"       # for the other requester's copy-out
        assert C.string_at(C.addressof(noted)).decode() == waits_first + (f"L{rank + 1}" if rank == 0 else "") + f"R{rank + 1}"
    for rank in range(2):
        assert L.bls_rank_complete(h, rank, C.c_int64(it), None, at(8), vp(rank + 1)) == 0
""")
