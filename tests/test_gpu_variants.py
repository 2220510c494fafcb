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


def layer(c, x, W, b, act=0):
    y = torch.full((x.shape[0], W.shape[0]), float("nan"), device=DEV)
    c.bls_mlp_layer(x, W, b, act, y)
    return y


def dense_ctx():
    import paper_2512_19342_amd as A
    return A.Context(1, 2, 4, 1, 4, [8] * 2, [0] * 2, A.BLS_FP32, 0)


# both sides of each line between the tiles (512 workgroups of 128 x 128, of 128 x 64) and a row per wavefront; sizes
# that no tile divides, steps of 16 and 32 k with and without a remainder
@pytest.mark.parametrize("M,K,N", [(65409, 33, 33), (65409, 415, 128), (32768, 64, 256), (65408, 16, 70), (32513, 45, 65),
                                   (16384, 31, 200), (16300, 8, 256), (4000, 129, 31), (257, 1, 5), (1029, 67, 4), (300, 130, 1)])
def test_layer_tiles(M, K, N):
    c = dense_ctx()
    g = torch.Generator(device=DEV).manual_seed(M + K)
    x, W, b = (torch.randn(s, device=DEV, generator=g) for s in ((M, K), (N, K), (N,)))
    y = layer(c, x, W, b)
    at = torch.unique(torch.cat([torch.arange(0, M, 61, device=DEV), torch.arange(max(0, M - 200), M, device=DEV)]))
    some = x[at].contiguous()
    assert torch.equal(layer(c, some, W, b), y[at])      # a sample's result does not depend on the others
    ref = some.double() @ W.double().t() + b.double()
    err = (K + 3) * 2.0 ** -24 * (some.abs().double() @ W.abs().double().t() + b.abs().double())
    assert bool(((y[at].double() - ref).abs() <= err).all())
    c.bls_check()


# what has no three bf16 parts, or parts outside the normal range
@pytest.mark.parametrize("M", [3, 70000])
def test_layer_infinities_and_the_ends_of_the_range(M):
    c = dense_ctx()
    K, N, inf, big = 40, 130, float("inf"), 3.4028234663852886e38
    x, W = torch.ones((M, K), device=DEV), torch.ones((N, K), device=DEV)
    x[0, 5], x[1, 7] = inf, float("nan")
    x[2] = 0.0
    x[2, 3] = big                                       # rounds up to the bf16 infinity
    x[M - 1, 9] = -inf
    W[:, 30] = torch.where(torch.arange(N, device=DEV) % 2 == 0, 1.0, 0.0)
    W[4, 5], W[6, 3] = 0.0, 0.5                         # inf * 0, big * 0.5
    W[7, 9] = inf                                       # a column that is infinite everywhere but where x is 0
    y = layer(c, x, W, None).cpu().double()
    ref = x.cpu().double() @ W.cpu().double().t()
    assert torch.equal(torch.isnan(y), torch.isnan(ref)) and torch.equal(torch.isinf(y), torch.isinf(ref))
    fin = torch.isfinite(ref)
    assert torch.equal(y[fin], ref[fin])                # small whole numbers and single products
    assert torch.equal(torch.sign(y[torch.isinf(y)]), torch.sign(ref[torch.isinf(ref)]))
    for ex, ew in ((-100, 90), (-116, 110), (110, -120), (60, 50)):
        g = torch.Generator(device=DEV).manual_seed(ex + 200)
        x = torch.randn((min(M, 300), K), device=DEV, generator=g)
        W = torch.randn((N, K), device=DEV, generator=g)
        one, scaled = layer(c, x, W, None), layer(c, x * 2.0 ** ex, W * 2.0 ** ew, None)
        # a part below 2^-126 may count as nothing: 2^-126 per value, against values of 2^ex and 2^ew
        loss = K * 4 * 4 * (2.0 ** (-126 - ex) + 2.0 ** (-126 - ew))
        assert bool(((scaled.double() * 2.0 ** -(ex + ew) - one.double()).abs() <= loss).all())


# layers of no, one, ... six whole steps of k, with and without a remainder, in each of the tiles
@pytest.mark.parametrize("M,N,step", [(65536, 65, 16), (32768, 127, 32), (190, 70, 32)])
def test_layer_steps(M, N, step):
    c = dense_ctx()
    for K in [1, *(n * step + d for n in range(1, 7) for d in (-1, 0, 1))]:
        g = torch.Generator(device=DEV).manual_seed(K)
        x, W, b = (torch.randn(s, device=DEV, generator=g) for s in ((M, K), (N, K), (N,)))
        y = layer(c, x, W, b)
        some, last = x[-150:].contiguous(), y[-150:]
        assert torch.equal(layer(c, some, W, b), last), K
        ref = some.double() @ W.double().t() + b.double()
        err = (K + 3) * 2.0 ** -24 * (some.abs().double() @ W.abs().double().t() + b.abs().double())
        assert bool(((last.double() - ref).abs() <= err).all()), K
    c.bls_check()


# the interaction's copy to LDS: more columns than threads, more pieces than a round of loads, one vector,
# odd lengths, whole tables and partial vectors; negative zeros among the values
@pytest.mark.parametrize("part,P,T,D,B", [(0, 3, 3, 479, 7), (1, 3, 3, 479, 7), (0, 2, 64, 200, 5), (1, 3, 64, 200, 5),
                                          (0, 1, 1, 4, 3), (1, 5, 1, 1, 9), (0, 4, 33, 100, 11), (1, 4, 26, 64, 33)])
def test_interaction_copies(part, P, T, D, B):
    c = permute_ctx(P, T, D, B, part)
    case = oracle.Case(P, T, D, B, part, [P * P] * T, [t % P for t in range(T)] if part == 0 else [0] * T, 0)
    rng = np.random.default_rng(T * D)
    S = rng.normal(size=c.n_vec * D).astype(np.float32)
    S[rng.random(S.size) < 0.1] = -0.0
    emb = oracle.unpack(case, oracle.exchange(case, S), None)
    x = rng.normal(size=(B, D)).astype(np.float32)
    dx, z, zs = (torch.from_numpy(x).to(DEV), *(torch.full((B, D + T * (T + 1) // 2), float("nan"), device=DEV) for _ in range(2)))
    c.bls_set_ring(torch.empty(c.n_vec * D, device=DEV))
    it, slot = c.bls_ring_advance()
    c.bls_alltoallv_local(torch.from_numpy(S).to(DEV), slot)
    c.bls_unpack_interact(it, dx, zs)
    c.bls_interact(dx, torch.from_numpy(emb).to(DEV), z)
    c.bls_check()
    ref, err = oracle.interact(x, emb)
    assert np.array_equal(zs.cpu().numpy().view(np.uint32), z.cpu().numpy().view(np.uint32))
    assert np.all(np.abs(z.cpu().numpy().astype(np.float64) - ref) <= err)
