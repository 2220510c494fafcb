"""The pooling kernels that keep a ring of rows in flight: the oracle's bits, and those of the kernels that take rows in
batches (64-bit and 32-bit positions), where a stream ends inside a ring or a block, in the shard's first and last rows, and for lookups
that have no row."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.test_gpu_parity import bits, case_of

pytestmark = pytest.mark.gpu

# lanes of a row: 4, 8, 16, 32, 64 (64: whole-wavefront groups), and rows whose last lanes idle
SHAPES = [("fp32", D) for D in (16, 32, 64, 100, 128, 256)] + [("fp16", D) for D in (32, 64, 128, 200, 512)] + [
    (dt, D) for dt in ("u8rq", "f8rq") for D in (64, 112, 128, 512)]
SHAPES += [("fp32", D) for D in (33, 62)] + [("fp16", D) for D in (36, 100, 180)] + [("u8rq", D) for D in (72, 100, 200)]   # wide groups of 4 and 8 bytes a lane
# rows of less than 64 bytes: four, eight and sixteen lanes of 4 or 8 bytes each, or one and two of 16 with few rows a segment
SHAPES += [("fp32", D) for D in (1, 2, 4, 5, 8, 10, 15)] + [("fp16", D) for D in (2, 8, 10, 16, 18, 20, 28)] + [
    (dt, D) for dt in ("u8rq", "f8rq") for D in (4, 16, 20, 32, 40, 60)]
BAGS = [(1, 1), (0, 3), (3, 9), (7, 17), (30, 70)]


def make(dt, D, part, bag):
    from paper_2512_19342_amd.runner import Pipeline
    w = synth.custom("ring", P=3, T=5, D=D, B=37, k=1, rows=[1, 2, 700, 33, 5], table_owner=[0, 1, 2, 0, 1] if part == 0 else None,
                     part_kind=part, bag=("uniform", *bag), table_dtype=dt, values="gauss", seed=D + bag[1], index_dist=("zipf", 1.1))
    tabs = [synth.make_table(w, t) for t in range(w.T)]       # row-wise, tables of one and two rows leave owners with none
    pipes = [Pipeline(w, [t.cuda() for t in tabs], 1 << 16) for _ in range(3)]
    pipes[1].ctx.bls_set_pool_tuning(wide_positions=1)
    pipes[2].ctx.bls_set_pool_tuning(wide_positions=0)        # the pool in batches with 32-bit positions
    return w, [t.numpy() for t in tabs], pipes


@pytest.mark.parametrize("bag", BAGS, ids=str)
@pytest.mark.parametrize("part", [0, 1], ids=["tables", "rows"])
@pytest.mark.parametrize("dt,D", SHAPES, ids=str)
def test_ring_adds_the_same_rows_in_the_same_order(dt, D, part, bag):
    w, tabs, pipes = make(dt, D, part, bag)
    ix, off = synth.make_batch(w, 0)
    nnz = int(off[-1])
    wts = torch.from_numpy(np.random.default_rng(nnz).uniform(-2.0, 2.0, size=nnz).astype(np.float32))
    for weights in (None, wts):
        ref = oracle.pipeline(case_of(w), tabs, ix.numpy(), off.numpy(), weights=None if weights is None else weights.numpy())
        for pipe in pipes:
            pipe.slots.fill_(float("nan"))
            if weights is None:
                j, slot = pipe.issue_fused(ix.cuda(), off.cuda(), nnz)
            else:
                j, slot = pipe.issue_weighted(ix.cuda(), off.cuda(), weights.cuda(), nnz, fused=True)
            assert (bits(pipe.slot_view(slot).cpu().numpy()) == bits(ref["R"].reshape(-1))).all()
            pipe.complete(j, pipe.new_out())
            pipe.ctx.bls_check()


@pytest.mark.parametrize("bag", BAGS[1:], ids=str)
@pytest.mark.parametrize("part", [0, 1], ids=["tables", "rows"])
@pytest.mark.parametrize("dt,D", [("fp32", D) for D in (16, 64, 100)] + [("fp16", D) for D in (32, 64, 128, 200, 512)] + [("u8rq", 64), ("u8rq", 128), ("f8rq", 128)], ids=str)
def test_streams_of_nine_segments(dt, D, part, bag):
    """Streams that a batch this small does not get by itself: blocks handed on and several ends of segments in a batch, with one store, with
    weights and, staged, with three."""
    w, tabs, pipes = make(dt, D, part, bag)
    ix, off = synth.make_batch(w, 4)
    nnz = int(off[-1])
    wts = torch.linspace(-1.0, 2.0, nnz)
    plain, weighted = (oracle.pipeline(case_of(w), tabs, ix.numpy(), off.numpy(), weights=x) for x in (None, wts.numpy()))
    for pipe, wide in zip(pipes, (-1, 1, 0)):
        pipe.ctx.bls_set_pool_tuning(segments_per_group=9, wide_positions=wide)
        for how, ref in (("fused", plain), ("weighted", weighted), ("staged", plain)):
            for buf in (pipe.pooled, pipe.send, pipe.slots):
                buf.fill_(float("nan"))
            if how == "fused":
                j, slot = pipe.issue_fused(ix.cuda(), off.cuda(), nnz)
            elif how == "weighted":
                j, slot = pipe.issue_weighted(ix.cuda(), off.cuda(), wts.cuda(), nnz, fused=True)
            else:
                j, slot = pipe.issue(ix.cuda(), off.cuda(), nnz)
                for k, buf in (("Y", pipe.pooled), ("S", pipe.send)):
                    assert (bits(buf.cpu().numpy()) == bits(ref[k].reshape(-1))).all(), (wide, k)
            assert (bits(pipe.slot_view(slot).cpu().numpy()) == bits(ref["R"].reshape(-1))).all(), (wide, how)
            pipe.complete(j, pipe.new_out())
        pipe.ctx.bls_check()


@pytest.mark.parametrize("width", [4, 8, 16])
@pytest.mark.parametrize("dt,D", [("fp32", 1), ("fp32", 2), ("fp32", 4), ("fp32", 8), ("fp16", 2), ("fp16", 8), ("fp16", 16), ("u8rq", 8), ("u8rq", 16),
                                  ("u8rq", 32), ("f8rq", 32)], ids=str)
def test_short_rows_by_chosen_lanes(dt, D, width):
    """Rows of at most 32 bytes with lanes of a width that the caller chose, some of them idle, with few and with many rows a segment."""
    for bag in ((0, 3), (7, 17)):
        w, tabs, pipes = make(dt, D, 1, bag)
        ix, off = synth.make_batch(w, 5)
        nnz = int(off[-1])
        ref = oracle.pipeline(case_of(w), tabs, ix.numpy(), off.numpy())
        for pipe, wide in zip(pipes, (-1, 1, 0)):
            pipe.ctx.bls_set_pool_tuning(lane_bytes=width, segments_per_group=3, wide_positions=wide)
            pipe.slots.fill_(float("nan"))
            j, slot = pipe.issue_fused(ix.cuda(), off.cuda(), nnz)
            assert (bits(pipe.slot_view(slot).cpu().numpy()) == bits(ref["R"].reshape(-1))).all(), (bag, wide)
            pipe.complete(j, pipe.new_out())
            pipe.ctx.bls_check()


@pytest.mark.parametrize("part", [0, 1], ids=["tables", "rows"])
@pytest.mark.parametrize("dt,D", [("fp32", 64), ("fp16", 128), ("u8rq", 64), ("f8rq", 128)], ids=str)
def test_lookups_without_a_row_add_nothing(dt, D, part):
    """Bad indices among good ones, their weights no numbers; infinities and NaN in the rows; sums that are exactly zero."""
    import paper_2512_19342_amd as B
    w, tabs, pipes = make(dt, D, part, (7, 17))
    if dt in ("fp32", "fp16"):
        for t in tabs:
            t[::3, ::5] = np.inf
            t[1::4, 1::7] = np.nan
            t[:, 2::5] = -0.0
        pipes = []
        for wide in (-1, 1, 0):
            from paper_2512_19342_amd.runner import Pipeline
            pipes.append(Pipeline(w, [torch.from_numpy(t).cuda() for t in tabs], 1 << 16))
            pipes[-1].ctx.bls_set_pool_tuning(wide_positions=wide)
    ix, off = synth.make_batch(w, 1)
    nnz = int(off[-1])
    wts = torch.linspace(-1.0, 2.0, nnz)
    table = torch.repeat_interleave(torch.arange(w.T).repeat_interleave(w.B), off[1:] - off[:-1])
    bad = torch.arange(nnz) % 5 == 2
    rows = torch.tensor(w.rows)[table]
    ix = torch.where(bad, torch.where(torch.arange(nnz) % 2 == 0, rows, torch.full_like(rows, -1)), ix)
    wts[bad] = torch.tensor([float("nan"), float("inf")])[torch.arange(int(bad.sum())) % 2]
    got = []
    for pipe in pipes:
        out = pipe.new_out()
        j, slot = pipe.issue_weighted(ix.cuda(), off.cuda(), wts.cuda(), nnz, fused=True)
        pipe.complete(j, out)
        with pytest.raises(B.BlsError):
            pipe.ctx.bls_check()
        plain = pipe.new_out()
        j, _ = pipe.issue_fused(ix.cuda(), off.cuda(), nnz)
        pipe.complete(j, plain)
        with pytest.raises(B.BlsError):
            pipe.ctx.bls_check()
        got.append((out.cpu().numpy(), plain.cpu().numpy()))
    good = ~bad
    goff = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(good, 0)])[off]
    want = [oracle.pipeline(case_of(w), tabs, ix[good].numpy(), goff.numpy(), weights=x)["Out"] for x in (wts[good].numpy(), None)]
    for g in got:
        for a, b in zip(g, want):
            assert (np.isnan(a) == np.isnan(b)).all()
            assert (bits(a)[~np.isnan(b)] == bits(b)[~np.isnan(b)]).all()


@pytest.mark.parametrize("bag", BAGS, ids=str)
@pytest.mark.parametrize("dt,D", [s for s in SHAPES if s[1] * {"fp32": 4, "fp16": 2}.get(s[0], 1) % 16 == 0], ids=str)
def test_one_launch_step_ring(dt, D, bag):
    """The one-launch step reads rows in a ring as well: every buffer, in either form of its positions, an index without a row
    among them."""
    import paper_2512_19342_amd as B
    w, tabs, pipes = make(dt, D, 0, bag)
    ix, off = synth.make_batch(w, 2)
    nnz = int(off[-1])
    ref = oracle.pipeline(case_of(w), tabs, ix.numpy(), off.numpy())
    for pipe in pipes:
        out = pipe.new_out().fill_(float("nan"))
        j = pipe.step_one_launch(ix.cuda(), off.cuda(), nnz, out)
        for k in ("ridx", "segoff", "sendcounts", "sdispls", "recvcounts", "rdispls"):
            assert (getattr(pipe, k).cpu().numpy()[:len(ref[k])] == ref[k]).all(), k
        for k, buf in (("Y", pipe.pooled), ("S", pipe.send), ("R", pipe.slot_view(j % pipe.ctx.K)), ("Out", out)):
            assert (bits(buf.cpu().numpy().reshape(-1)) == bits(ref[k].reshape(-1))).all(), k
        pipe.ctx.bls_check()
    at = nnz // 2
    bad = ix.clone()
    bad[at] = -1
    goff = off.clone()
    goff[goff > at] -= 1
    want = oracle.pipeline(case_of(w), tabs, np.delete(ix.numpy(), at), goff.numpy())["Out"]
    for pipe in pipes:
        out = pipe.new_out()
        pipe.step_one_launch(bad.cuda(), off.cuda(), nnz, out)
        with pytest.raises(B.BlsError):
            pipe.ctx.bls_check()
        assert (bits(out.cpu().numpy()) == bits(want)).all()


@pytest.mark.parametrize("dt,D", [("fp32", 16), ("fp32", 64), ("fp16", 64), ("fp16", 256), ("u8rq", 16), ("u8rq", 128), ("f8rq", 64)], ids=str)
def test_bags_past_the_lookups_are_empty(dt, D):
    """A run edge that lies past the next one makes the runs longer than the lookups there are: the bags that no longer fit are
    empty, whatever their neighbours of the same wavefront still have, and the error is raised."""
    import paper_2512_19342_amd as B
    w, tabs, pipes = make(dt, D, 0, (3, 9))
    ix, off = synth.make_batch(w, 3)
    nnz, n = int(off[-1]), w.B
    past = 11                                                 # table 2 starts behind table 3
    boff = off.clone()
    boff[2 * n] = int(off[3 * n]) + past
    outs = []
    for pipe in pipes:
        out = pipe.new_out().fill_(float("nan"))
        j = pipe.step_one_launch(ix.cuda(), boff.cuda(), nnz, out)
        with pytest.raises(B.BlsError) as e:
            pipe.ctx.bls_check()
        assert e.value.code == B.BLS_ERANGE
        outs.append([t.cpu().numpy().reshape(-1).copy() for t in (pipe.pooled, pipe.send, pipe.slot_view(j % pipe.ctx.K), out)])
        starts = pipe.segoff.cpu().numpy()[:w.T * n + 1]      # in the send order
    assert starts[-1] > nnz                                   # what the runs add up to
    for a, *others in zip(*outs):
        assert all((bits(a) == bits(b)).all() for b in others)
    over = (starts[1:] > nnz) & (starts[1:] > starts[:-1])
    assert over.any() and not over.all()
    for S in (o[1] for o in outs):
        assert not S.reshape(-1, D)[over].any() and S.reshape(-1, D)[~over].any()


@pytest.mark.parametrize("rows", [8388599, 8388600], ids=["the largest shard of a ring", "one row more"])
def test_shards_that_end_where_32_bit_offsets_do(rows):
    """Rows of 512 bytes on both sides of 2 GB and at the shard's end, one and twelve a bag, and an index just past it."""
    import paper_2512_19342_amd as B
    from types import SimpleNamespace
    from paper_2512_19342_amd.runner import Pipeline
    P, n = 2, 64
    tab = torch.zeros(rows, 128, device="cuda")
    at = torch.tensor([0, 1, 4194303, 4194304, rows // 2, rows - 2, rows - 1])
    vals = torch.from_numpy(np.random.default_rng(rows).standard_normal((len(at), 128)).astype(np.float32))
    tab[at.cuda()] = vals.cuda()
    w = SimpleNamespace(P=P, T=1, D=128, k=1, B=n, rows=[rows], table_owner=[1], table_dtype="fp32", part_kind=B.BLS_TABLE_WISE)
    pipe = Pipeline(w, [tab], 12 * n)
    for per in (1, 12):
        pick = torch.from_numpy(np.random.default_rng(per).integers(0, len(at), n * per))
        off = torch.arange(n + 1) * per
        want = np.zeros((n, 128), np.float32)
        for j in range(per):
            want += vals[pick.view(n, per)[:, j]].numpy()
        out = pipe.new_out()
        j, _ = pipe.issue_fused(at[pick].cuda(), off.cuda(), n * per)
        pipe.complete(j, out)
        pipe.ctx.bls_check()
        assert (bits(out.cpu().numpy().reshape(n, 128)) == bits(want)).all(), per
        pipe.step_one_launch(at[pick].cuda(), off.cuda(), n * per, out)
        pipe.ctx.bls_check()
        assert (bits(out.cpu().numpy().reshape(n, 128)) == bits(want)).all(), per
    past = torch.full((n,), rows)
    j, _ = pipe.issue_fused(past.cuda(), torch.arange(n + 1).cuda(), n)
    pipe.complete(j, out)
    with pytest.raises(B.BlsError):
        pipe.ctx.bls_check()
    assert not out.any()
