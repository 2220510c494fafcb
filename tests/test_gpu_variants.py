"""Kernel variants chosen by size, type or alignment, at the sizes where the choice changes, against
the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def permute_ctx(P, T, D, B, part):
    """A context whose permutes can run: shards of P rows, never read."""
    import paper_2512_19342_amd as A
    c = A.Context(P, T, D, 1, B, [P * P] * T, [t % P for t in range(T)], A.BLS_FP32, part)
    tab = torch.zeros((P * P, (D + 3) // 4 * 4), device=DEV)
    for t in range(T):
        for d in range(P):
            n = c.bls_shard_range(t, d)[1]
            if n:
                c.bls_set_shard(t, d, tab[:n])
    c.desc = torch.empty(c.bls_desc_bytes(), dtype=torch.uint8, device=DEV)
    c.bls_commit(c.desc)
    return c


# one vector short of and at the 96 MB from which the permutes stream, rows of 16-byte pieces and odd ones,
# mini-batches of unequal size
@pytest.mark.parametrize("part,P,T,D,B", [(0, 3, 12, 128, 16383), (0, 3, 12, 128, 16384), (1, 3, 4, 128, 16383),
                                          (1, 3, 4, 128, 16384), (0, 5, 8, 97, 32430), (0, 5, 8, 97, 32431),
                                          (1, 4, 2, 97, 32430), (1, 4, 2, 97, 32431)])
@pytest.mark.parametrize("mean", [False, True])
def test_permutes_on_both_sides_of_the_streaming_size(part, P, T, D, B, mean):
    c = permute_ctx(P, T, D, B, part)
    case = oracle.Case(P, T, D, B, part, [P * P] * T, [t % P for t in range(T)] if part == 0 else [0] * T, 0)
    rng = np.random.default_rng(B)
    Y = rng.normal(size=c.n_vec * D).astype(np.float32)
    offsets = np.concatenate([[0], np.cumsum(rng.integers(0, 5, T * B))]).astype(np.int64)
    S, R = torch.empty(c.n_vec * D, device=DEV), torch.empty(c.n_vec * D, device=DEV)
    out = torch.empty((B, T, D), device=DEV)
    c.bls_set_ring(R)
    c.bls_pack(torch.from_numpy(Y).to(DEV), S)
    it, slot = c.bls_ring_advance()
    c.bls_alltoallv_local(S, slot)
    if mean:
        c.bls_unpack_mean(it, torch.from_numpy(offsets).to(DEV), out)
    else:
        c.bls_unpack(it, out)
    c.bls_check()
    s = oracle.pack(case, Y)
    r = oracle.exchange(case, s)
    assert np.array_equal(S.cpu().numpy().view(np.uint32), s.view(np.uint32))
    assert np.array_equal(R.cpu().numpy().view(np.uint32), r.view(np.uint32))
    ref = oracle.unpack(case, r, offsets if mean else None)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))
