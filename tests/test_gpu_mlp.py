"""bls_mlp against bls_mlp_layer, layer by layer: the same bits in the same rows, nothing else touched, nothing launched
when a layer is refused."""
import pytest
import torch

from tests.test_gpu_dense import DEV, ctx_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,rows", [(1, None), (70, None), (70, (0, 70)), (70, (13, 0)), (70, (13, 40)), (300, (255, 45))])
@pytest.mark.parametrize("widths", [(13,), (13, 5), (13, 512, 256, 64), (415, 130, 64, 1), (7, 1, 1)])
def test_layers_in_one_call(M, rows, widths):
    import paper_2512_19342_amd as A
    c = ctx_for(2, 4, 4)
    g = torch.Generator(device=DEV).manual_seed(M)
    x = torch.randn(M, widths[0], device=DEV, generator=g)
    net = [(torch.randn(n, k, device=DEV, generator=g), torch.randn(n, device=DEV, generator=g) if i != 1 else None,
            A.BLS_ACT_RELU if i + 2 < len(widths) else A.BLS_ACT_SIGMOID)
           for i, (k, n) in enumerate(zip(widths, widths[1:]))]
    lo, n = (0, M) if rows is None else rows
    more = 0 if rows is None else 3                           # outputs may be longer than the rows that are asked for
    ys = [torch.full((M + more, W.shape[0]), -7.0, device=DEV) for W, _, _ in net]
    c.bls_mlp(x, [(W, b, act, y) for (W, b, act), y in zip(net, ys)], rows)
    a = x[lo:lo + n]
    for (W, b, act), y in zip(net, ys):
        want = torch.empty(n, W.shape[0], device=DEV)
        c.bls_mlp_layer(a, W, b, act, want)
        assert torch.equal(y[lo:lo + n], want)
        assert bool((y[:lo] == -7).all()) and bool((y[lo + n:] == -7).all())
        a = want


def test_a_refused_layer_launches_nothing():
    import paper_2512_19342_amd as A
    c = ctx_for(2, 4, 4)
    x, W = torch.ones(4, 4, device=DEV), torch.ones(4, 4, device=DEV)
    ys = [torch.zeros(4, 4, device=DEV) for _ in range(2)]
    with pytest.raises(A.BlsError) as e:
        c.bls_mlp(x, [(W, None, A.BLS_ACT_RELU, ys[0]), (W, None, 7, ys[1])])
    assert e.value.code == A.BLS_EINVAL
    c.bls_check()
    assert bool((ys[0] == 0).all())
    for bad in ((-1, 2), (0, 5), (3, 2)):
        with pytest.raises(AssertionError):
            c.bls_mlp(x, [(W, None, A.BLS_ACT_RELU, ys[0])], bad)
    with pytest.raises(AssertionError):
        c.bls_mlp(x, [(W[:, :3], None, A.BLS_ACT_RELU, ys[0])])
    with pytest.raises(AssertionError):
        c.bls_mlp(x, [(W, None, A.BLS_ACT_RELU, torch.zeros(5, 4, device=DEV))])
