"""Layers in tiles of 64 x 64, whose wavefronts either split or multiply: edges of the tiles, steps that end inside a
chunk of eight k or a step of 32, and the same bits as the larger tiles give a sample among many."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_dense import DEV, ctx_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(1, 65), (63, 100), (64, 128), (65, 129), (200, 70)])
@pytest.mark.parametrize("K", [1, 7, 8, 9, 16, 31, 32, 33, 40, 63, 64, 65, 95, 96, 97, 129, 415])
def test_small_tiles(M, N, K):
    c = ctx_for()
    rng = np.random.default_rng(M * 1000 + K)
    x = rng.normal(size=(M, K)).astype(np.float32)
    W = (rng.normal(size=(N, K)) / np.sqrt(K)).astype(np.float32)
    b = rng.normal(size=N).astype(np.float32)
    xd, Wd, bd = (torch.from_numpy(a).to(DEV) for a in (x, W, b))
    y = torch.full((M + 1, N), -7.0, device=DEV)
    c.bls_mlp_layer(xd, Wd, bd, 1, y[:M])
    ref, err = oracle.mlp_layer(x, W, b, 1)
    assert np.all(np.abs(y[:M].cpu().numpy() - ref) <= err)   # the oracle's bound: (K + 3) roundings
    assert bool((y[M] == -7).all())
    many = 128 * 512                                          # two larger tiles and more for every compute unit
    big = torch.zeros(many, K, device=DEV)
    big[:M] = xd
    yb = torch.empty(many, N, device=DEV)
    c.bls_mlp_layer(big, Wd, bd, 1, yb)
    assert torch.equal(yb[:M], y[:M])
    bad = xd.clone()
    bad[M - 1, K - 1] = float("nan")
    y2 = torch.empty(M, N, device=DEV)
    c.bls_mlp_layer(bad, Wd, None, 0, y2)
    assert bool(torch.isnan(y2[M - 1]).all()) and bool(torch.isfinite(y2[:M - 1]).all())
