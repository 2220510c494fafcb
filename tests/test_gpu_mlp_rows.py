"""DenseModel's rows: what slices of the tensors take (whole numbers of any kind, a range that ends past the batch, one row of
a tensor whose rows are apart), layer by layer as bls_mlp_layer gives it, and nothing else touched."""
import numpy as np
import pytest
import torch

from tests.test_gpu_dense import DEV, ctx_for

pytestmark = pytest.mark.gpu
T, D, B, K = 2, 8, 40, 13


def make():
    from paper_2512_19342_amd.runner import DenseModel
    c = ctx_for(T, D, B)
    g = torch.Generator(device=DEV).manual_seed(3)
    net = lambda widths: [(torch.randn(n, k, device=DEV, generator=g), torch.randn(n, device=DEV, generator=g)) for k, n in zip(widths, widths[1:])]
    m = DenseModel(c, net((K, 20, D)), net((D + T * (T + 1) // 2, 6, 1)), B)
    return c, m, torch.rand(B, K, device=DEV, generator=g), torch.randn(B, T, D, device=DEV, generator=g)


def expect(c, a, layers, acts):
    for (W, b), act in zip(layers, acts):
        y = torch.empty(a.shape[0], W.shape[0], device=DEV)
        c.bls_mlp_layer(a.contiguous(), W, b, act, y)
        a = y
    return a


@pytest.mark.parametrize("rows", [(7, 9), (np.int64(7), np.int32(9)), (np.int64(0), B), np.array([7, 9]), [7, 9], (B - 3, 5), (B, 4), (12, 0)],
                         ids=lambda r: f"{type(r).__name__}-{r[0]}-{r[1]}")
def test_bottom_takes_what_a_slice_takes(rows):
    import paper_2512_19342_amd as A
    c, m, dense, _ = make()
    lo, hi = int(rows[0]), min(int(rows[0]) + int(rows[1]), B)
    out = torch.full((B, D), -7.0, device=DEV)
    assert m.apply_bottom(dense, out, rows=rows) is out
    c.bls_check()
    assert torch.equal(out[lo:hi], expect(c, dense[lo:hi], m.bottom, [A.BLS_ACT_RELU] * 2))
    assert bool((out[:lo] == -7).all()) and bool((out[hi:] == -7).all())


@pytest.mark.parametrize("rows", [(7, 9), (np.int64(7), np.int32(9))])
def test_prediction_of_some_rows(rows):
    import paper_2512_19342_amd as A
    c, m, dense, emb = make()
    lo, hi = 7, 16
    x = m.apply_bottom(dense).clone()
    z, p = torch.empty_like(m.z), torch.full((B, 1), -7.0, device=DEV)
    c.bls_interact(x, emb, z)
    assert m.compute_ctr(x, emb, p, rows=rows) is p
    assert torch.equal(p[lo:hi], expect(c, z[lo:hi], m.top, [A.BLS_ACT_RELU, A.BLS_ACT_SIGMOID]))
    assert bool((p[:lo] == -7).all()) and bool((p[hi:] == -7).all())


def test_one_row_of_tensors_whose_rows_are_apart():
    import paper_2512_19342_amd as A
    c, m, dense, _ = make()
    wide_in, wide_out = torch.full((B, K + 3), -7.0, device=DEV), torch.full((B, D + 5), -7.0, device=DEV)
    wide_in[:, :K] = dense
    m.apply_bottom(wide_in[:, :K], wide_out[:, :D], rows=(11, 1))
    assert torch.equal(wide_out[11:12, :D], expect(c, dense[11:12], m.bottom, [A.BLS_ACT_RELU] * 2))
    wide_out[11, :D] = -7.0
    assert bool((wide_out == -7).all())
    with pytest.raises(AssertionError):
        m.apply_bottom(wide_in[:, :K], None, rows=(11, 2))


def test_list_of_layers_with_numpy_rows():
    import paper_2512_19342_amd as A
    c, m, dense, _ = make()
    (W, b), out = m.bottom[0], torch.full((B, 20), -7.0, device=DEV)
    c.bls_mlp(dense, [(W, b, A.BLS_ACT_RELU, out)], (np.int64(5), np.int64(6)))
    assert torch.equal(out[5:11], expect(c, dense[5:11], m.bottom[:1], [A.BLS_ACT_RELU]))
    assert bool((out[:5] == -7).all()) and bool((out[11:] == -7).all())
