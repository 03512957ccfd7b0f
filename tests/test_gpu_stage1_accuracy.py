"""Accuracy of the binary64 stage against double-double vectors."""
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def zk():
    import torch
    import paper_2402_11868_amd as Z
    return Z, Z.Context(), torch


@pytest.mark.parametrize("n", [130, 300, 512])
def test_rounding_of_the_rank_two_updates(zk, n):
    """|x_i^H v_j| |lam_i - lam_j| / ||H|| of neighbouring eigenvalues is the
    backward error in that place.  An entry of a random matrix is about
    ||H|| / (2 sqrt n), a rounding 0.4 u of it, the trailing blocks hold a third
    of the entries: k roundings a column for n columns put 0.4 u sqrt(k n / 3)
    / (2 sqrt n) = 0.115 u sqrt(k) there.  Four (each product added to the
    entry by itself) are 0.23 u, beside what the tridiagonal solver leaves,
    which falls with 1 / sqrt n; a reduction whose entries keep their rounding
    errors stays below 0.18 u from order 300 on."""
    Z, ctx, torch = zk
    tot = 0.0
    for seed in (1, 2):
        g = torch.Generator().manual_seed(seed * 77 + n)
        x = 2.0 * torch.rand((2, n, n), generator=g, dtype=torch.float64) - 1.0
        h = torch.complex(x[0], x[1])
        h = (h + h.mH).cuda()
        r, = Z.heev_allpairs(ctx, [[h]])
        (w, V), = Z.heev_fp64(ctx, [h])
        M = (r.V[0].mH @ V).abs()
        lam = r.w[0]
        gap = (lam[1:] - lam[:-1]) / float(lam.abs().max())
        tot += float(((torch.diagonal(M, 1) * gap) ** 2 + (torch.diagonal(M, -1) * gap) ** 2).mean()) / 4
    assert tot ** 0.5 <= (0.18 if n >= 300 else 0.27) * U
