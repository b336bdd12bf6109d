"""Input estimation at the ends of its tiles: 64 block columns and 32 pairs to
a matrix-instruction tile, 8 blocks to a response, 16 pairs to a norm, shares
with and without room for their partial results; and a silent pair."""
import numpy as np
import pytest
import torch

from oracle import inversion as inv
from oracle import misfit as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


# 4 x blocks columns: 4, 64 (a full tile), 68, 132, 260; pairs 3 .. 258; a
# short record of many blocks leaves no room for partial results
@pytest.mark.parametrize("n_rec,stride,blocks,shifts", [(1, 1, 1, 1), (1, 3, 16, 5), (11, 5, 17, 17), (5, 7, 33, 9),
                                                        (86, 2, 65, 40), (2, 2, 40, 3), (16, 1, 9, 8)])
def test_fit_matches_oracle(sw, n_rec, stride, blocks, shifts):
    rng = np.random.default_rng(n_rec + blocks)
    n = stride * blocks
    G = [rng.standard_normal((n, n_rec, 3)) for _ in range(3)]
    c = rng.standard_normal((3, shifts))
    obs = sum(c[j, l] * np.concatenate([np.zeros((l * stride, n_rec, 3)), G[j][:n - l * stride]]) for j in range(3)
              for l in range(shifts))
    obs = obs + 0.1 * rng.standard_normal(obs.shape)
    if n_rec > 1:
        obs[:, 1, 2] = 0.0  # silent: carries no weight
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = sw.Context(0)
    got_c, err, used, rank, U = sw.fit_input(ctx, [dev(g) for g in G], dev(obs), stride, shifts, return_response=True)
    assert used == 3 * n_rec - (n_rec > 1)
    assert err == pytest.approx(om.err(U.cpu().numpy(), obs)[0], rel=1e-12, abs=1e-12)
    want = np.asarray(inv.fit(G, obs, stride, shifts)[0]).reshape(3, shifts)
    resp = lambda x: sum(x[j, l] * np.concatenate([np.zeros((l * stride, n_rec, 3)), G[j][:n - l * stride]])
                         for j in range(3) for l in range(shifts))
    assert np.allclose(U.cpu().numpy(), resp(got_c), rtol=0, atol=1e-12 * np.abs(obs).max())
    # the objective's residual is what the coefficients are for: equal to the
    # oracle's to the square of the solution's error (kept condition <= 1e6)
    w = inv.pair_weights(obs)
    J = lambda x: float((w * ((resp(x) - obs) ** 2).sum(0)).sum())
    assert J(got_c) <= J(want) * (1 + 1e-9) + 1e-12
