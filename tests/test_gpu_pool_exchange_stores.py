"""bls_embbag_pool_exchange by the form its stores take (storage, rows a segment, length of a vector): the bits of the four
calls in all three buffers, into a ring slot and, behind another stream's copy-out, without it."""
import pytest
import torch

import oracle
import synth
from tests.test_gpu_parity import bits, case_of
from tests.test_gpu_pool_exchange import make

pytestmark = pytest.mark.gpu

# (storage, D, bags): 16 floats a lane; eight of long vectors, few rows a segment (plain) and more; four and eight of vectors
# that share 64-byte pieces, short and long; fewer than four
SHAPES = [(dt, D, bag) for dt in ("u8rq", "f8rq") for D in (64, 112, 256) for bag in ((1, 1), (0, 9))]
SHAPES += [("fp16", D, bag) for D in (128, 256, 272, 264, 512) for bag in ((0, 1), (0, 2), (2, 6))] + [("u8rq", 264, (0, 2))]
SHAPES += [("fp32", D, (0, 7)) for D in (20, 28, 36, 60, 68, 132, 34, 33)] + [("fp16", D, (0, 7)) for D in (24, 40, 56, 72, 136, 100, 66, 64)]
SHAPES += [("u8rq", D, (0, 7)) for D in (72, 136, 100)]


@pytest.mark.parametrize("part", [0, 1], ids=["tables", "rows"])
@pytest.mark.parametrize("dt,D,bag", SHAPES, ids=lambda v: str(v))
def test_same_bits_whatever_the_stores(dt, D, bag, part):
    w = synth.custom("stores", P=3, T=5, D=D, B=67, k=1, rows=[40, 300, 7, 90, 1001], table_owner=[0, 1, 2, 0, 1] if part == 0 else None,
                     part_kind=part, bag=("uniform", *bag),
                     table_dtype=dt, values="gauss", seed=D, index_dist=("zipf", 1.1))
    pipe, tabs = make(w)
    other = torch.cuda.Stream()
    for it, on in enumerate((None, other, None)):
        ix, off = synth.make_batch(w, it)
        ref = oracle.pipeline(case_of(w), tabs, ix.numpy(), off.numpy())
        for buf in (pipe.pooled, pipe.send, pipe.slots) if it == 0 else (pipe.pooled, pipe.send):
            buf.fill_(float("nan"))
        j, slot = pipe.issue(ix.cuda(), off.cuda(), int(off[-1]))
        for name, t in (("Y", pipe.pooled), ("S", pipe.send), ("R", pipe.slot_view(slot))):
            assert (bits(t.cpu().numpy()) == bits(ref[name].reshape(-1))).all(), (name, it)
        out = pipe.new_out()
        pipe.complete(j, out, on)
        torch.cuda.synchronize()
        assert (bits(out.cpu().numpy()) == bits(ref["Out"])).all(), it
    pipe.ctx.bls_check()
