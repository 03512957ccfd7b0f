"""Storage of a session's requests: a request that is done gives its iterates
back, whatever else was admitted with it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_done_requests_give_their_storage_back():
    import torch
    import paper_2402_11868_amd as Z

    ctx = Z.Context()
    rng = np.random.default_rng(3)
    a = rng.uniform(-1, 1, (500, 500)) + 1j * rng.uniform(-1, 1, (500, 500))
    slow = torch.from_numpy(a + a.conj().T).cuda()          # takes two rounds
    fast = torch.from_numpy(W.householder_hermitian(np.linspace(-1.0, 1.0, 128), seed=2)).cuda()   # one round
    s = Z.Session(ctx)
    # the first request keeps the scheduler busy while the others queue, so that they are admitted together
    tickets = [s.submit([slow])]
    late = s.submit([slow])
    quick = [s.submit([fast]) for _ in range(120)]
    for t in quick:
        assert s.result(t).status == Z.ZK_OK
    # what is given back later, when the slow ones are done, is their own iterates (4 planes of 500^2
    # doubles each); the quick ones had 63 MB.  (The engine's plans only grow while the session lives.)
    held = ctx.memory()["transient"]
    for t in tickets + [late]:
        assert s.result(t).status == Z.ZK_OK
    assert held - ctx.memory()["transient"] <= 2 * (8 * 4 * 500 * 500 + 8 * 2 * 500 + 512)
    s.close()
    assert ctx.memory()["transient"] == 0
    ctx.close()
