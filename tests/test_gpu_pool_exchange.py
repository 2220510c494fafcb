"""bls_embbag_pool_exchange against the four calls it stands for: every buffer, the ring and the errors."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.test_gpu_parity import EDGE, bits, case_of

pytestmark = pytest.mark.gpu

SHAPES = [synth.workload(1), synth.workload(3, "small"), synth.workload(4, "small"), synth.workload(5, "small")] + [
    synth.custom("edge", k=2, values="gauss", table_dtype=dt, seed=53, index_dist=("zipf", 1.1), **e)
    for e in EDGE for dt in ("fp32", "fp16", "u8rq", "f8rq")]


def make(w, k=None):
    from paper_2512_19342_amd.runner import Pipeline
    if k is not None:
        w.k = k
    tabs = [synth.make_table(w, t) for t in range(w.T)]
    return Pipeline(w, [t.cuda() for t in tabs], 1 << 21), [t.numpy() for t in tabs]


@pytest.mark.parametrize("w", SHAPES, ids=lambda w: f"{w.name}-{w.table_dtype}-D{w.D}-P{w.P}-B{w.B}")
def test_one_launch_leaves_what_the_four_calls_leave(w):
    pipe, tabs = make(w)
    c, case = pipe.ctx, case_of(w)
    for it in range(3):
        ix, off = synth.make_batch(w, it)
        nnz = int(off[-1])
        ref = oracle.pipeline(case, tabs, ix.numpy(), off.numpy())
        for buf in (pipe.pooled, pipe.send, pipe.slots):
            buf.fill_(float("nan"))
        j, slot = pipe.issue(ix.cuda(), off.cuda(), nnz)
        assert (j, slot) == (it, it % c.K) and c.bls_ring_state()[:2] == (it + 1, it)
        got = [t.clone() for t in (pipe.pooled, pipe.send, pipe.slot_view(slot))]
        for name, g in zip(("Y", "S", "R"), got):
            assert np.array_equal(bits(g.cpu().numpy()), bits(ref[name].reshape(-1))), (name, it)
        out = pipe.new_out()
        pipe.complete(j, out)
        assert np.array_equal(bits(out.cpu().numpy()), bits(ref["Out"])), it
        c.bls_embbag_pool(pipe.ridx, pipe.segoff, nnz, pipe.pooled)
        c.bls_pack(pipe.pooled, pipe.send)
        assert torch.equal(pipe.pooled.view(torch.int32), got[0].view(torch.int32))
        assert torch.equal(pipe.send.view(torch.int32), got[1].view(torch.int32))
    c.bls_check()


@pytest.mark.parametrize("k", [1, 3])
def test_completion_on_another_stream(k):
    """The slot is refilled only after the copy-out that another stream still runs; every output as the oracle's."""
    w = synth.workload(4, "small")
    pipe, tabs = make(w, k)
    case, other = case_of(w), torch.cuda.Stream()
    done, pending = [], []
    for it in range(6):
        ix, off = synth.make_batch(w, it)
        if len(pending) == pipe.ctx.K:
            pipe.ctx.bls_rank_delay(300, other)                   # the copy-out starts late
            j, out = pending.pop(0)
            pipe.complete(j, out, other)
        j, _ = pipe.issue(ix.cuda(), off.cuda(), int(off[-1]))
        pending.append((j, pipe.new_out()))
        done.append((pending[-1][1], oracle.pipeline(case, tabs, ix.numpy(), off.numpy())["Out"]))
    for j, out in pending:
        pipe.complete(j, out, other)
    torch.cuda.synchronize()
    for it, (out, ref) in enumerate(done):
        assert np.array_equal(bits(out.cpu().numpy()), bits(ref)), it
    pipe.ctx.bls_check()


def test_a_full_ring_is_refused_after_pool_and_pack():
    import paper_2512_19342_amd as B
    w = synth.workload(4, "small")
    pipe, tabs = make(w, 1)
    batches = [synth.make_batch(w, it) for it in range(2)]
    first, _ = pipe.issue(batches[0][0].cuda(), batches[0][1].cuda(), int(batches[0][1][-1]))
    with pytest.raises(B.BlsError) as e:
        pipe.issue(batches[1][0].cuda(), batches[1][1].cuda(), int(batches[1][1][-1]))
    assert e.value.code == B.BLS_ERING_FULL
    ref = [oracle.pipeline(case_of(w), tabs, ix.numpy(), off.numpy()) for ix, off in batches]
    assert np.array_equal(bits(pipe.pooled.cpu().numpy()), bits(ref[1]["Y"].reshape(-1)))
    assert np.array_equal(bits(pipe.send.cpu().numpy()), bits(ref[1]["S"].reshape(-1)))
    out = pipe.new_out()
    pipe.complete(first, out)                                     # the first iteration's slot is untouched
    assert np.array_equal(bits(out.cpu().numpy()), bits(ref[0]["Out"]))
    pipe.ctx.bls_check()


def test_argument_errors():
    import paper_2512_19342_amd as B
    w = synth.workload(1)
    pipe, _ = make(w)
    ix, off = synth.make_batch(w, 0)
    nnz = int(off[-1])
    c = pipe.ctx
    c.bls_plan(ix.cuda(), off.cuda(), nnz, pipe.sendcounts, pipe.sdispls, pipe.recvcounts, pipe.rdispls, pipe.ridx, pipe.segoff,
               None, pipe.ws)
    for bad in (dict(ridx=None), dict(segoff=None), dict(nnz=-1), dict(pooled=None), dict(send=None), dict(send=pipe.pooled),
                dict(send=pipe.send[1:])):
        args = dict(ridx=pipe.ridx, segoff=pipe.segoff, nnz=nnz, pooled=pipe.pooled, send=pipe.send)
        with pytest.raises(B.BlsError) as e:
            c.bls_embbag_pool_exchange(**{**args, **bad})
        assert e.value.code == B.BLS_EINVAL and c.bls_ring_state()[:2] == (0, 0)
