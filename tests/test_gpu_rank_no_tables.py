"""Per-rank iterations where some ranks own no table: they put nothing and complete their samples all the same."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.test_gpu_parity import bits, case_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 4, 7])                     # streams, one segment a group, rows of single floats
@pytest.mark.parametrize("owner", [[0, 0], [2, 1], [2, 2]])
def test_ranks_without_tables(owner, D):
    from paper_2512_19342_amd.runner import Pipeline
    w = synth.custom("bare", P=3, T=2, D=D, B=50, k=2, rows=[90, 40], part_kind=0, table_owner=owner, values="gauss", bag=("uniform", 0, 5))
    tabs = [synth.make_table(w, t) for t in range(w.T)]
    pipe = Pipeline(w, [t.cuda() for t in tabs], 1 << 16)
    streams = [torch.cuda.Stream() for _ in range(w.P)]
    for it in range(4):
        ix, off = synth.make_batch(w, it)
        nnz = int(off[-1])
        pipe.ctx.bls_plan(ix.cuda(), off.cuda(), nnz, pipe.sendcounts, pipe.sdispls, pipe.recvcounts, pipe.rdispls, pipe.ridx, pipe.segoff,
                          None, pipe.ws)
        torch.cuda.synchronize()
        out = torch.full((w.B, w.T, w.D), float("nan"), device="cuda")
        for r in range(w.P):
            pipe.ctx.bls_rank_put(r, pipe.ridx, None, pipe.segoff, nnz, it, streams[r])
        for r in range(w.P):
            pipe.ctx.bls_rank_complete(r, it, None, out, streams[r])
        torch.cuda.synchronize()
        ref = oracle.pipeline(case_of(w), [t.numpy() for t in tabs], ix.numpy(), off.numpy())["Out"]
        assert np.array_equal(bits(out.cpu().numpy()), bits(ref)), it
    pipe.ctx.bls_check()
