"""Sums over the times of records (misfit, norms of the input estimation) at
the numbers of pairs where another width serves them, and at lengths around a
workgroup's times; and no slower with a few long records than with many short
ones of the same size."""
import time

import numpy as np
import pytest
import torch

from oracle import misfit as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


# pairs 3 .. 24: one a workgroup; 27 .. 300: 4; 303 .. 1500: 8; more: 16
@pytest.mark.parametrize("n_rec", [1, 8, 9, 100, 101, 500, 501, 700])
@pytest.mark.parametrize("n", [1, 63, 257, 1025])
def test_misfit(sw, n_rec, n):
    rng = np.random.default_rng(n_rec + n)
    obs = rng.standard_normal((n, n_rec, 3))
    U = obs + 0.3 * rng.standard_normal(obs.shape)
    if n_rec > 1:
        obs[:, n_rec // 2, 1] = 0.0              # silent
    ctx = sw.Context(0)
    err, used = sw.misfit(ctx, torch.from_numpy(U), torch.from_numpy(obs))
    assert used == 3 * n_rec - (n_rec > 1)
    # sums of up to 1025 squares in another order
    assert err == pytest.approx(om.err(U, obs)[0], rel=2e-13)


def test_few_long_records(sw):
    """The two sums of 6 pairs by 200000 steps and of 1200 by 1000: the same
    bytes, and a few long records have a work-item for every 1024th value."""
    ctx = sw.Context(0)
    t = {}
    for n_rec, n in ((2, 200000), (400, 1000)):
        g = torch.Generator("cuda").manual_seed(1)
        U, obs = (torch.randn(n, n_rec, 3, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
        best = []
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sw.misfit(ctx, U, obs)
            best.append(time.perf_counter() - t0)
        t[n_rec] = min(best)
    print(t)
    # 16 pairs a workgroup: one workgroup, 3125 steps a work-item; a pair a
    # workgroup: 195.  The call's fixed cost (30 us) on both sides.
    assert t[2] <= 10 * t[400]
