"""Which kernel a call launches, and on how many workgroups, without a GPU: the few HIP runtime calls are replaced by a library
that notes the launches, and the kernels' names as the library registers them."""
from tests import test_exchange_host as host

NAMES = r"""
static const void *known[2048];
static const char *called[2048];
static int n_known;
void __hipRegisterFunction(void **m, const void *f, char *d, const char *name, unsigned l, void *a, void *b, void *c, void *e, int *w)
{
    if (n_known < 2048) { known[n_known] = f; called[n_known++] = name; }
}
char kernel[1024];                      /* of the latest launch, as the compiler spells it */
unsigned grid_x, lds_bytes;
static void look(const void *f, unsigned x, size_t sh)
{
    const char *s = "?";
    for (int i = 0; i < n_known; ++i) if (known[i] == f) s = called[i];
    int k = 0;
    while (s[k] && k < 1023) { kernel[k] = s[k]; ++k; }
    kernel[k] = 0;
    grid_x = x;
    lds_bytes = (unsigned)sh;
}
int hipLaunchKernel("""

LOOK = r"""
import re, subprocess
x, y, lds = (C.c_uint.in_dll(stub, n) for n in ("grid_x", "grid_y", "lds_bytes"))
def kernel():                                                 # "pool_stream<16, 0, ...>"
    name = C.string_at(C.addressof(C.c_char.in_dll(stub, "kernel")))
    name = subprocess.run(["c++filt"], input=name, capture_output=True).stdout.decode().replace("(anonymous namespace)::", "")
    return re.match(r"(?:void )?([^<(]*(?:<.*?>(?=\())?)", name)[1]
def config(P, T, D, B, dtype=0, part=0, rows=9, k=1):
    h = vp()
    assert L.bls_create(C.byref(Config(P, T, D, k, B, dtype, part, (C.c_int64 * T)(*[rows] * T), (C.c_int32 * T)(*[t % P for t in range(T)]))), C.byref(h)) == 0
    for t in range(T):
        for d in [t % P] if part == 0 else range(P):
            a, n = C.c_int64(), C.c_int64()
            assert L.bls_shard_range(h, t, d, C.byref(a), C.byref(n)) == 0
            if n.value: assert L.bls_set_shard(h, t, d, at(1), n) == 0
    n = C.c_size_t()
    assert L.bls_desc_bytes(h, C.byref(n)) == 0 and L.bls_commit(h, at(2), n, None) == 0
    assert L.bls_set_ring(h, at(3), C.c_size_t(1 << 44)) == 0
    return h
def pool(h, nnz, weighted=False):
    rc = L.bls_embbag_pool_weighted(h, at(4), at(5), at(6), C.c_int64(nnz), at(7), None) if weighted else L.bls_embbag_pool(h, at(4), at(5), C.c_int64(nnz), at(7), None)
    assert rc == 0
    return kernel()
def plan(h, nnz):
    stub.forget()
    assert L.bls_plan(h, at(4), at(5), C.c_int64(nnz), at(6), at(7), at(8), at(9), at(10), at(11), None, at(12), C.c_size_t(1 << 40), None) == 0
    return C.string_at(C.addressof(noted)).decode().count("L")
def step(h, nnz):
    assert L.bls_step_tablewise(h, at(4), at(5), C.c_int64(nnz), at(6), at(7), at(8), at(9), at(10), at(11), None, at(13), at(14), at(15), None, None) == 0
    return kernel()
"""


def run(tmp_path, monkeypatch, body):
    runtime = host.RUNTIME.replace("int hipLaunchKernel(", NAMES).replace("grid_y = g.y;", "grid_y = g.y; look(f, g.x, sh);")
    assert runtime.count("look(") == 2
    monkeypatch.setattr(host, "RUNTIME", runtime)
    return host.run(tmp_path, LOOK + body)


def test_a_runs_workgroups_in_a_plan_of_one_launch(tmp_path, monkeypatch):
    """Tables differ in their bags, and a run's workgroups copy all of it: past 2^22 lookups a run gets no fewer of them than the
    three launches give it, below about four thousand in all."""
    run(tmp_path, monkeypatch, r"""
for P, T, B, nnz in ((8, 32, 16384, 8_900_000), (2, 64, 16384, 7_600_000), (8, 26, 16384, 5_700_000), (8, 32, 16384, 10 << 20), (1, 4, 40000, 8_100_000),
                     (1, 300, 64, 1 << 22), (8, 32, 4096, 1 << 22), (4, 26, 2048, 53248), (8, 200, 512, 1 << 20)):
    h = config(P, T, 16, B)
    runs = P * T
    assert L.bls_set_plan_tuning(h, 0) == 0 and plan(h, nnz) == 3 and kernel() == "plan_place_runs"
    three = x.value
    assert L.bls_set_plan_tuning(h, -1) == 0 and plan(h, nnz) == 1 and kernel() == "plan_runs_one_launch" and y.value == runs
    assert x.value >= (three if nnz > 1 << 22 else min(three, -(-4096 // runs))), (P, T, B, nnz, x.value, three)
for P, T, nnz, launches in ((8, 32, (10 << 20) + 1, 3), (1, 300, (1 << 22) + 1, 3), (8, 300, 1 << 20, 3)):
    h = config(P, T, 16, 4096)
    assert plan(h, nnz) == launches, (P, T, nnz)
""")


def test_the_one_launch_step_takes_short_bags_in_batches(tmp_path, monkeypatch):
    """Either side of every line: rows a bag by storage and lanes, workgroups, and shards at the end of 32-bit offsets."""
    run(tmp_path, monkeypatch, r"""
fp32, fp16, u8, f8 = 0, 1, 2, 3
for dtype, D, lanes, rows in ((fp32, 128, 32, 16), (fp32, 20, 8, 16), (fp32, 16, 4, 3), (fp32, 8, 2, 0), (fp32, 4, 1, 0), (fp16, 64, 8, 13), (fp16, 200, 32, 13),
                              (fp16, 32, 4, 3), (fp16, 16, 2, 0), (u8, 128, 8, 1 << 20), (f8, 112, 8, 1 << 20), (u8, 512, 32, 1 << 20), (u8, 64, 4, 3), (f8, 32, 2, 0)):
    # one workgroup more than the chip holds at once, as many as that, one more than there are compute units
    for P, T, B, rows in ((1, 1, 7 * 256 * (256 // lanes) + 1, rows), (1, 1, 7 * 256 * (256 // lanes), min(rows, 6)), (1, 1, 256 * (256 // lanes) + 1, min(rows, 6))):
        h = config(P, T, D, B, dtype)
        for nnz, batch in ((rows * T * B, "false"), (rows * T * B - 1, "true"), (T * B if rows > 1 else 0, "true" if rows else "false")):
            if nnz < 0: continue
            assert step(h, nnz) == f"step_tablewise<{lanes}, {dtype}, {batch}>", (dtype, D, P, nnz, kernel())
            for tuned, batch in ((0, "false"), (1, "true")):
                assert L.bls_set_pool_tuning(h, 0, 0, -1, tuned) == 0 and step(h, nnz) == f"step_tablewise<{lanes}, {dtype}, {batch}>"
            assert L.bls_set_pool_tuning(h, 0, 0, -1, -1) == 0
    h = config(1, 1, D, 256 * (256 // lanes), dtype)
    assert step(h, 1) == f"step_tablewise<{lanes}, {dtype}, false>"
for rows, batch in ((0xfffff000 // 512 - 1, "false"), (0xfffff000 // 512, "true")):
    h = config(2, 2, 128, 64, fp32, rows=rows)
    assert step(h, 6400) == f"step_tablewise<32, 0, {batch}>", rows
""")


def test_the_pools_ring_by_rows_a_segment(tmp_path, monkeypatch):
    """Either side of every line: storage, weights, rows a segment, megabytes of vectors."""
    run(tmp_path, monkeypatch, r"""
fp32, fp16, u8, f8 = 0, 1, 2, 3
for dtype, weighted, small, large in ((fp32, False, 2, 8), (fp32, True, 1, 2), (fp16, False, 4, 8), (fp16, True, 2, 4), (u8, False, 6, 12), (f8, True, 6, 12)):
    for mb, rows in ((1, small), (96, small), (97, large), (999, large)):
        B = (mb << 20) // (8 * 128 * 4)
        h = config(2, 8, 128, B, dtype)
        for nnz, ring_ in ((rows * 8 * B, "true"), (rows * 8 * B - 1, "false")):
            name = pool(h, nnz, weighted)
            assert name.startswith(f"pool_stream<{ {fp32: 32, fp16: 16}.get(dtype, 8)}, {dtype}, 16, "), name
            assert name.endswith(f" false, {str(weighted).lower()}, {ring_}, 0>"), (dtype, weighted, mb, rows, name)
""")


def test_positions_and_the_ring_can_be_chosen_apart(tmp_path, monkeypatch):
    """wide_positions 0: the loop in batches with 32-bit positions, which the library takes for shards from 4 GB on (up to 64 GB with
    lanes of 16 bytes) and where the ring does not pay."""
    run(tmp_path, monkeypatch, r"""
for rows, own, zero in ((9, "false, false, true", "false, false, false"), (0xfffff000 // 512, "false, false, false", "false, false, false"),
                        (0xffffffff // 32 + 1, "true, false, false", "true, false, false")):
    h = config(2, 8, 128, 64, rows=rows)
    for tuned, form in ((-1, own), (0, zero), (1, "true, false, false")):
        assert L.bls_set_pool_tuning(h, 0, 0, -1, tuned) == 0
        assert pool(h, 8 * 64 * 32) == f"pool_stream<32, 0, 16, 8, {form}, 0>", (rows, tuned, kernel())
        rc, it, slot, calls = issue(h, 0, 8 * 64 * 32)
        assert rc == 0 and calls == "L0R0" and kernel() == f"pool_stream<32, 0, 16, 8, {form}, 3>", kernel()
        assert unpack(h, it, 0)[0] == 0
""")


def test_lane_bytes_are_what_was_asked_for(tmp_path, monkeypatch):
    """Rows that one or two lanes of 16 bytes cover are split over four narrower ones by the library, not where the caller chose a
    width.  Widths that do not divide a row are halved until they do."""
    run(tmp_path, monkeypatch, r"""
fp32, fp16, u8, f8 = 0, 1, 2, 3
for dtype, D, few, many, widths in ((fp16, 8, (1, 16), (4, 4), {16: (1, 16), 8: (4, 8), 4: (4, 4)}), (fp32, 8, (2, 16), (4, 8), {16: (2, 16), 8: (4, 8), 4: (8, 4)}),
                                    (u8, 16, (1, 16), (4, 4), {16: (1, 16), 8: (4, 8), 4: (4, 4)}), (f8, 32, (4, 8), (4, 8), {16: (2, 16), 8: (4, 8), 4: (8, 4)}),
                                    (fp32, 2, (4, 4), (4, 4), {16: (4, 8), 8: (4, 8), 4: (4, 4)}), (fp32, 64, (16, 16), (16, 16), {16: (16, 16), 8: (32, 8), 4: (64, 4)}),
                                    (fp16, 10, (8, 4), (8, 4), {16: (8, 4), 8: (8, 4), 4: (8, 4)})):
    h = config(2, 4, D, 64, dtype, rows=1 << 21)
    for rows, free in ((5, few), (6, many)):
        for chosen, (lanes, vb) in ((0, free), *widths.items()):
            assert L.bls_set_pool_tuning(h, chosen, 0, -1, -1) == 0
            name = pool(h, rows * 4 * 64)
            assert name.startswith(f"pool_{'stream' if lanes >= 4 else 'rows'}<{lanes}, {dtype}, {vb}, "), (dtype, D, rows, chosen, name)
""")


def test_a_ring_is_held_to_four_workgroups_with_long_segments(tmp_path, monkeypatch):
    """LDS that nothing uses, from twelve rows a segment on; fewer rows, 32 and 64 lanes of 4 bytes, shards that an XCD's L2 holds, and
    batches ask for none."""
    run(tmp_path, monkeypatch, r"""
fp32, fp16, u8, f8 = 0, 1, 2, 3
for dtype, D, held in ((fp32, 128, True), (fp32, 16, True), (fp32, 6, True), (fp32, 8, True), (fp32, 17, False), (fp32, 33, False), (fp16, 64, True), (fp16, 20, True), (fp16, 50, False),
                       (fp16, 100, True), (u8, 128, True), (u8, 32, True), (u8, 60, True), (u8, 100, False), (f8, 24, True)):
    row = D * 4 if dtype == fp32 else D * 2 if dtype == fp16 else (D + 8 + 15) // 16 * 16
    h = config(2, 8, D, 512, dtype, rows=(4 << 20) // row)
    assert "true" in pool(h, 99 * 8 * 512) and lds.value == 0
    h = config(2, 8, D, 512, dtype, rows=(4 << 20) // row + 1)
    for nnz in (3 * 8 * 512, 12 * 8 * 512 - 1, 12 * 8 * 512, 99 * 8 * 512):
        for weighted in (False, True):
            name = pool(h, nnz, weighted)
            in_ring = name.startswith("pool_stream<") and name.endswith("true, 0>")
            assert in_ring or nnz < 12 * 8 * 512, (dtype, D, name)
            assert lds.value == (36 * 1024 if in_ring and held and nnz >= 12 * 8 * 512 else 0), (dtype, D, nnz, name, lds.value)
            assert L.bls_set_pool_tuning(h, 0, 0, -1, 0) == 0 and not pool(h, nnz, weighted).endswith("true, 0>") and lds.value == 0
            assert L.bls_set_pool_tuning(h, 0, 0, -1, -1) == 0
""")


def test_few_shards_are_dealt_where_one_xcds_l2_holds_them(tmp_path, monkeypatch):
    """One store: rows of 512 bytes and more, of shards of 1.5 to 8 MB, with four rows a segment, are dealt to the XCDs from 55 % of them at work
    on, all others from 70 %."""
    run(tmp_path, monkeypatch, r"""
for D, rows, size, line in ((128, 4, 2 << 20, 55), (128, 4, (3 << 19) + 512, 55), (128, 4, 3 << 19, 70), (128, 40, 8 << 20, 55), (128, 8, (8 << 20) + 512, 70), (128, 3, 2 << 20, 70),
                            (64, 8, 2 << 20, 70), (256, 8, 2 << 20, 55), (128, 40, 50 << 20, 70)):
    for T in (1, 4, 5, 6, 8, 9, 10, 11, 12, 16, 17, 40):
        B = (20 << 20) // (T * 512)
        h = config(1, T, D, B, rows=size // (4 * D))
        assert pool(h, rows * T * B).startswith(f"pool_stream<{D // 4}, 0, 16, 8, ")
        assert y.value == (1 if 100 * T >= line * 8 * ((T + 7) // 8) else T), (D, rows, size, T, y.value)
""")


def test_short_rows_take_four_lanes_where_they_pay(tmp_path, monkeypatch):
    """Either side of every line: one and two lanes of 16 bytes, shards that the caches hold, megabytes of vectors, rows a segment."""
    run(tmp_path, monkeypatch, r"""
fp32, fp16, u8, f8 = 0, 1, 2, 3
never = 1 << 40
for dtype, D, lanes, lines in ((fp32, 8, 2, ((16, never, never), (6, 6, 8))), (fp16, 16, 2, ((16, never, never), (6, 6, 8))), (fp32, 4, 1, ((6, 12, 16), (6, 6, 6))),
                               (fp16, 8, 1, ((6, 12, 16), (6, 6, 6))), (u8, 16, 1, ((6, 6, 16), (6, 6, 6))), (f8, 16, 1, ((6, 6, 16), (6, 6, 6)))):
    row = D * 4 if dtype == fp32 else D * 2 if dtype == fp16 else (D + 8 + 15) // 16 * 16
    for size, by_mb in zip((4 << 20, (4 << 20) + row), lines):
        for mb, line in zip((20, 60, 400), by_mb):
            B = (mb << 20) // (4 * D * 4)
            h = config(2, 4, D, B, dtype, rows=size // row)
            for nnz in (4 * B, min(line, 99) * 4 * B - 1, min(line, 99) * 4 * B):
                four = nnz >= line * 4 * B
                assert pool(h, nnz).startswith(f"pool_stream<4, {dtype}, " if four else f"pool_rows<{lanes}, {dtype}, 16, "), (dtype, D, size, mb, nnz / (4 * B), kernel())
for mb in (20, 400):
  B = (mb << 20) // (4 * 32 * 4)
  for size in (4 << 20, 5 << 20):
    h = config(2, 4, 32, B, u8, rows=size // 48)
    for rows in (1, 3, 4, 15, 16):
        four = mb == 20 or rows < 4 or (rows >= 16 and size > 4 << 20)
        assert pool(h, rows * 4 * B).startswith("pool_stream<4, 2, 8, " if four else "pool_rows<2, 2, 16, "), (mb, rows, kernel())
""")
