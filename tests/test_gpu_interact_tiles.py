"""The interaction in tiles of 16 x 16 at its edges, and the shapes that keep the tiles of 32 x 32."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_dense import DEV, ctx_for

pytestmark = pytest.mark.gpu


# vectors around multiples of 16, one step of k and several; 900 x 16 fits LDS only in rows without padding
@pytest.mark.parametrize("T,D", [(1, 16), (15, 16), (16, 48), (17, 128), (31, 32), (32, 112), (33, 64), (63, 128), (64, 16), (65, 96),
                                 (100, 32), (129, 16), (900, 16), (30, 256), (16, 24), (33, 17)])
@pytest.mark.parametrize("shift", [0, 1])                     # floats the vectors start off a 16-byte boundary
def test_tiles_match_the_oracle(T, D, shift):
    B = 9
    rng = np.random.default_rng(T * 7 + D)
    x, emb = rng.normal(size=(B, D)).astype(np.float32), rng.normal(size=(B, T, D)).astype(np.float32)
    room = torch.empty(B * T * D + shift, device=DEV)
    room[shift:] = torch.from_numpy(emb.reshape(-1))
    z = torch.full((B, D + T * (T + 1) // 2), float("nan"), device=DEV)
    c = ctx_for(T, D, B)
    c.bls_interact(torch.from_numpy(x).to(DEV), room[shift:], z)
    c.bls_check()
    ref, err = oracle.interact(x, emb)
    got = z.cpu().numpy()
    assert np.array_equal(got[:, :D], x)
    assert np.all(np.abs(got - ref) <= err)


def test_a_vector_that_is_not_finite_stays_in_its_own_products():
    T, D, B = 40, 32, 6
    x, emb = torch.randn(B, D, device=DEV), torch.randn(B, T, D, device=DEV)
    clean = torch.empty(B, D + T * (T + 1) // 2, device=DEV)
    c = ctx_for(T, D, B)
    c.bls_interact(x, emb, clean)
    emb[2, 17, 5] = float("nan")
    z = torch.empty_like(clean)
    c.bls_interact(x, emb, z)
    i, j = torch.tril_indices(T + 1, T + 1, -1)
    hit = torch.zeros_like(clean, dtype=torch.bool)
    hit[2, D:] = ((i == 18) | (j == 18)).to(DEV)
    assert torch.isnan(z[hit]).all() and torch.equal(z[~hit], clean[~hit])
