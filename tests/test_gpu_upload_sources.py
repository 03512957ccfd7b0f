"""Calls that upload their tables twice with no wait between (an FP32 start of
order-1 matrices has nothing to project) and calls that fail after an upload:
the sources of enqueued copies stay untouched until the copies are done."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import torch
    import paper_2402_11868_amd as Z
    return Z, torch


def test_fp32_start_of_order_one(zk):
    Z, torch = zk
    ctx = Z.Context()
    rng = np.random.default_rng(1)
    for count in (3000, 1, 700, 2999):
        d = rng.standard_normal(count)
        mats = [[torch.full((1, 1), complex(x), dtype=torch.complex128, device="cuda")] for x in d]
        res = Z.heev(ctx, mats, opts=Z.make_opts(init_fp32=True))
        assert [r.status for r in res] == [Z.ZK_OK] * count
        assert np.array_equal(np.array([float(r.w[0][0]) for r in res]), d)
    ctx.close()


def test_calls_that_run_out_of_room(zk):
    """A refused call, at whatever point, leaves the context as it was."""
    Z, torch = zk
    mats = [[torch.from_numpy(W.householder_hermitian(np.linspace(-1.0, 1.0, n), seed=n)).cuda()] for n in (40, 90, 7, 64)]
    free = Z.Context()
    want = Z.heev(free, mats)
    refused = 0
    for kib in range(512, 8192, 384):
        ctx = Z.Context(0, budget=kib << 10)
        for _ in range(2):
            try:
                got = Z.heev(ctx, mats)
            except RuntimeError as e:
                assert "ENOMEM" in str(e)
                refused += 1
                continue
            for g, a in zip(got, want):
                for x, y in zip(list(g.w) + list(g.V), list(a.w) + list(a.V)):
                    assert torch.equal(x, y)
        assert ctx.memory()["transient"] == 0
        ctx.close()
    assert refused > 0
    free.close()
