"""The binary64 stage on matrices far from norm 1: a power of two in the input
is the same power of two in the eigenvalues and nothing in the vectors."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import torch
    import paper_2402_11868_amd as Z
    return Z, Z.Context(), torch


@pytest.mark.parametrize("n", [2, 40, 128, 130, 300])
def test_power_of_two(zk, n):
    # 2^-505: squares of entries near 1e-152 are normal numbers, but their sum over a column lies below 2^-1000;
    # 2^505: they stay below the overflow threshold
    Z, ctx, torch = zk
    g = torch.Generator().manual_seed(n)
    x = 2.0 * torch.rand((2, n, n), generator=g, dtype=torch.float64) - 1.0
    h = torch.complex(x[0], x[1])
    h = (h + h.mH).cuda()
    (w, V), = Z.heev_fp64(ctx, [h])
    assert float((h @ V - V * w).abs().max()) <= 10 * n * 2.0 ** -53 * float(w.abs().max())
    for e in (-505, -60, 60, 505):
        (ws, Vs), = Z.heev_fp64(ctx, [h * 2.0 ** e])
        assert torch.equal(ws * 2.0 ** -e, w), e
        assert torch.equal(Vs, V), e

