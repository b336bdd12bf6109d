"""The operator passes where their tables and tiles end: material tables
longer than a workgroup (loaded in several rounds), tiles at their caps, and a
capped grid (a workgroup walks several tiles)."""
import numpy as np
import pytest
import torch

import casegen as cg
from oracle import march

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


def _rel(a, b):
    return float(torch.linalg.norm(a.double() - b.double()) / torch.linalg.norm(b.double()))


# 85 materials fill the first round of 256 work-items, 86 start a second; 255 is the most
@pytest.mark.parametrize("n_mat", [85, 86, 171, 255])
def test_long_material_tables(sw, n_mat):
    """A table that repeats two materials gives the two-material operator."""
    ctx = sw.Context(0)
    mesh = cg.box_mesh(40.0, 40.0, 40.0, 5.0, jitter=0.2)
    gm = sw.Mesh(ctx, mesh)
    case = cg.make_case(mesh, cg.CONFIGS["small"], n_steps=3, n_rec=2)
    two = {p: sw.Case(ctx, gm, case, precision=p, guess="poly") for p in ("fp64", "mixed")}
    rng = np.random.default_rng(n_mat)
    ids = np.arange(n_mat)
    case.mat = case.mat[ids % 2].copy()
    pick = [ids[ids % 2 == k] for k in (0, 1)]
    case.tet_mat = np.where(case.tet_mat == 0, rng.choice(pick[0], mesh.n_tets), rng.choice(pick[1], mesh.n_tets)).astype(np.uint8)
    many = {p: sw.Case(ctx, gm, case, precision=p, guess="poly") for p in ("fp64", "mixed")}
    x = torch.from_numpy(rng.standard_normal(3 * mesh.n_nodes)).cuda()
    # the same arithmetic: only the arrival order of the additions differs
    for op in ("A", "M", "K", "M+K+Cabs"):
        assert _rel(many["fp64"].apply(op, x), two["fp64"].apply(op, x)) < 1e-14
        assert _rel(many["mixed"].apply_f32(op, x), two["mixed"].apply_f32(op, x)) < 1e-6
    u, v, a = (rng.standard_normal(3 * mesh.n_nodes) for _ in range(3))
    for c in (two["fp64"], many["fp64"]):
        c.set_state(u, v, a)
    assert _rel(many["fp64"].rhs(), two["fp64"].rhs()) < 1e-14
    for p in ("fp64", "mixed"):
        for c in (two[p], many[p]):
            c.set_state(u * 1e-3, v * 1e-3, a * 1e-3)
            c.step(3)
        assert np.linalg.norm(many[p].waveforms() - two[p].waveforms()) <= 1e-6 * np.linalg.norm(two[p].waveforms())


@pytest.mark.parametrize("nodes,elems", [(1280, 1024), (1280, 511), (64, 16), (300, 257)])
@pytest.mark.parametrize("cap", [0, 8, 16])
def test_tile_sizes_and_capped_grids(sw, nodes, elems, cap):
    ctx = sw.Context(0)
    mesh = cg.box_mesh(50.0, 40.0, 40.0, 5.0, jitter=0.2)
    case = cg.make_case(mesh, cg.CONFIGS["small"], n_steps=2, n_rec=2)
    ctx.set_grid_cap(cap)
    gm = sw.Mesh(ctx, mesh, tile_nodes=nodes, tile_elems=elems)
    s = march.build_system(mesh, case)
    A = march.step_matrix(s, case.dt)
    x = np.random.default_rng(1).standard_normal(3 * mesh.n_nodes)
    ref = torch.from_numpy(A @ x).cuda()
    xd = torch.from_numpy(x).cuda()
    gc = sw.Case(ctx, gm, case, precision="mixed")
    assert _rel(gc.apply("A", xd), ref) < 1e-13
    ref32 = torch.from_numpy(A @ x.astype(np.float32).astype(np.float64)).cuda()
    assert _rel(gc.apply_f32("A", xd), ref32) < 1e-6
    # right-hand side b = F + M (4/dt v + a) + C v - K u
    u, v, a = (np.random.default_rng(k).standard_normal(3 * mesh.n_nodes) for k in (2, 3, 4))
    gc.set_state(u, v, a)
    rhs = case.v_in[1] @ s.Fb + s.M @ (4.0 / case.dt * v + a) + s.C @ v - s.K @ u
    assert _rel(gc.rhs(), torch.from_numpy(rhs).cuda()) < 1e-13
    b = sw.Batch(ctx, [gc, sw.Case(ctx, gm, case, precision="mixed")])
    for y in b.apply_f32([xd, xd]):
        assert _rel(y, ref32) < 1e-6
