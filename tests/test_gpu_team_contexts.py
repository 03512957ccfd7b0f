"""Several contexts on one GPU whose teams of the resident tridiagonalisation
need more compute units together than there are: their launches follow one
another, none gives up, and every result is the one of a call alone."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def _mat(torch, n, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((2, n, n), generator=g, dtype=torch.float64)
    h = torch.complex(x[0], x[1])
    return (h + h.mH).cuda()


@pytest.mark.parametrize("orders", [(1100, 1300), (900, 1000, 1030, 700), (200, 64, 400, 1024)])
def test_threads(orders):
    import torch
    import paper_2402_11868_amd as Z

    ctxs = [Z.Context() for _ in orders]
    mats = [_mat(torch, n, n) for n in orders]
    alone = [Z.heev_fp64(c, [m])[0] for c, m in zip(ctxs, mats)]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        try:
            for _ in range(4):
                (w, V), = Z.heev_fp64(ctxs[k], [mats[k]])
                if not (torch.equal(w, alone[k][0]) and torch.equal(V, alone[k][1])):
                    bad.append(("bits", k))
        except Exception as e:   # noqa: BLE001
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(orders))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    assert all(c.team_stats()["gave_up"] == 0 for c in ctxs)
    for c in ctxs:
        c.close()
    # a new context after the last holder of the gate is gone
    c = Z.Context()
    (w, V), = Z.heev_fp64(c, [mats[0]])
    assert torch.equal(w, alone[0][0]) and torch.equal(V, alone[0][1])
    c.close()
