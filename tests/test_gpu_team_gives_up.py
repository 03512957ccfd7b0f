"""The resident tridiagonalisation when its work-groups do not come together:
the waits are bounded, every kernel ends, and the per-column launches reduce
the matrices that gave up.  The bound is set to nothing from the host."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture
def zk(monkeypatch):
    import torch
    import paper_2402_11868_amd as Z
    plain = Z.Context()
    monkeypatch.setenv("ZK_TRD_WAIT_US", "0")
    ctx = Z.Context()
    yield Z, torch, plain, ctx
    ctx.close()
    plain.close()


def _mat(torch, n, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((2, n, n), generator=g, dtype=torch.float64)
    q, _ = torch.linalg.qr(torch.complex(x[0], x[1]))
    h = (q * torch.linspace(-1.0, 1.0, n, dtype=torch.float64)) @ q.mH
    return 0.5 * (h + h.mH)


@pytest.mark.parametrize("n", [129, 300, 600, 1100])
def test_alone(zk, n):
    Z, torch, plain, ctx = zk
    H = _mat(torch, n, n)
    (w, V), = Z.heev_fp64(ctx, [H.cuda()])
    assert ctx.team_stats() == {"matrices": 1, "gave_up": 1}
    # the backward error of a Householder reduction and inverse iteration: a modest multiple of n u ||H||, ||H|| = 1
    Hd = H.cuda()
    assert float((Hd @ V - V * w).abs().max()) <= 10 * n * U
    assert float((w.cpu() - torch.linalg.eigvalsh(H)).abs().max()) <= 10 * n * U
    Z.heev_fp64(plain, [Hd])
    assert plain.team_stats() == {"matrices": 1, "gave_up": 0}


def test_some_of_a_call(zk):
    """Matrices that need no team keep their bits; the others are the per-column ones."""
    Z, torch, plain, ctx = zk
    orders = [64, 130, 1, 128, 300, 2]
    mats = [_mat(torch, n, 9 + n).cuda() for n in orders]
    got = Z.heev_fp64(ctx, mats)
    assert ctx.team_stats() == {"matrices": 2, "gave_up": 2}
    for n, m, (w, V) in zip(orders, mats, got):
        (wa, Va), = Z.heev_fp64(ctx if n > 128 else plain, [m])
        assert torch.equal(w, wa) and torch.equal(V, Va), n


def test_refinement_and_refused_input(zk):
    Z, torch, plain, ctx = zk
    H = torch.from_numpy(W.householder_hermitian(W.spectrum_c4(160), seed=3)).cuda()
    for call in (lambda c: Z.heev(c, [[H]])[0], lambda c: Z.heev_allpairs(c, [[H]])[0]):
        r, a = call(ctx), call(plain)
        assert r.status == Z.ZK_OK
        # both within the gate of 1e-30 ||H||, so of each other within twice that
        d = (r.w[0] - a.w[0]) + (r.w[1] - a.w[1])
        assert float(d.abs().max()) <= 2e-30 * float(a.w[0].abs().max())
        assert max(i["resid"] for i in r.info) <= 1e-30 * float(a.w[0].abs().max())
    assert ctx.team_stats()["gave_up"] >= 2
    bad = _mat(torch, 200, 1)
    bad[150, 20] = float("nan")
    with pytest.raises(RuntimeError, match="ZK_EINVAL"):
        Z.heev_fp64(ctx, [bad.cuda()])


def test_without_allocation(zk):
    Z, torch, plain, ctx = zk
    H = torch.from_numpy(W.householder_hermitian(W.spectrum_c4(200), seed=5)).cuda()
    r, = Z.heev(ctx, [[H]], noalloc=True)
    a, = Z.heev(ctx, [[H]])
    assert r.status == Z.ZK_OK and ctx.team_stats()["gave_up"] >= 2
    for x, y in zip(list(r.w) + list(r.V), list(a.w) + list(a.V)):
        assert torch.equal(x, y)
