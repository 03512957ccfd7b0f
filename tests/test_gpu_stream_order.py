"""Inputs that are still being written on torch's current stream when an entry
point is called, and outputs of the call before that are still being read:
every call gives the bits of a call on finished inputs."""
import pytest

pytestmark = pytest.mark.gpu


def _herm(torch, n, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((2, n, n), generator=g, dtype=torch.float64)
    h = torch.complex(x[0], x[1])
    return (h + h.mH).cuda()


def _calls(Z, torch):
    def eig(r):
        return list(r.w) + list(r.V)

    def fp64(ctx, h):
        (w, V), = Z.heev_fp64(ctx, [h])
        return [w, V]

    def svd(ctx, h):
        r, = Z.svd(ctx, [h[:, :30]])
        return [r.s, r.U, r.V]

    def refine(ctx, h):
        (w, V), = Z.heev_fp64(ctx, [h])
        return eig(Z.rqi_refine(ctx, [h], w, V, 2))

    def session(ctx, h):
        s = Z.Session(ctx)
        r = s.result(s.submit([h]))
        s.close()
        return eig(r)

    def two_site(ctx, h):
        n = h.shape[0] // 2 * 2
        r = Z.mps_two_site(ctx, h[:n, :16] / 64, h[:16, :n] / 64, torch.eye(4, dtype=h.dtype, device=h.device), chi_max=32)
        return [r.A, r.s, r.B]

    return {
        "heev": lambda c, h: eig(Z.heev(c, [[h]])[0]),
        "heev_two_planes": lambda c, h: eig(Z.heev(c, [[h, h * 2.0 ** -60]])[0]),
        "noalloc": lambda c, h: eig(Z.heev(c, [[h]], noalloc=True)[0]),
        "qd": lambda c, h: eig(Z.heev(c, [[h]], limbs_out=4)[0]),
        "allpairs": lambda c, h: eig(Z.heev_allpairs(c, [[h]])[0]),
        "mp": lambda c, h: eig(Z.heev_mp(c, [[h]], limbs=8)[0]),
        "fp64": fp64, "svd": svd, "refine": refine, "session": session, "two_site": two_site,
    }


NAMES = ["heev", "heev_two_planes", "noalloc", "qd", "allpairs", "mp", "fp64", "svd", "refine", "session", "two_site"]


@pytest.mark.parametrize("own_stream", [False, True])
@pytest.mark.parametrize("name", NAMES)
def test_pending_inputs(name, own_stream):
    import torch
    import paper_2402_11868_amd as Z

    ctx = Z.Context(stream=torch.cuda.Stream() if own_stream else None)
    call = _calls(Z, torch)[name]
    h, other = _herm(torch, 48, 1), _herm(torch, 48, 2)
    torch.cuda.synchronize()
    want = call(ctx, h)
    torch.cuda.synchronize()
    for _ in range(2):
        torch.cuda._sleep(20_000_000)     # some ms on torch's stream before the input is there
        late = torch.empty_like(h).copy_(h)
        got = call(ctx, late)
        torch.cuda._sleep(20_000_000)
        read = [x * 1.0 for x in got]     # still reading when the next call runs
        del got
        call(ctx, other)
        torch.cuda.synchronize()
        for x, y in zip(read, want):
            assert torch.equal(x, y)
    ctx.close()


@pytest.mark.parametrize("n,count", [(150, 4), (304, 4), (572, 1)])
def test_passes_that_nothing_waits_between(n, count):
    import torch
    import paper_2402_11868_amd as Z

    ctx = Z.Context()
    a = [_herm(torch, n, k) for k in range(count)]
    b = [_herm(torch, n, 50 + k) for k in range(count)]
    ref = _herm(torch, n, 99)[0]

    def run(mats):
        out = Z.heev_fp64(ctx, mats)
        return torch.stack([w for w, _ in out]), torch.stack([V * torch.sgn(ref @ V).conj() for _, V in out])

    want = run(a)
    torch.cuda.synchronize()
    for _ in range(5):
        run(a)
        run(b)
        got = run(a)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    ctx.close()
