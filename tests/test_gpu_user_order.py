"""Operator passes that read and write the user's node order, against the
passes between copies in the internal order, which serve a call whose output
overlaps its input; nodes of no tile and guard values around the output."""
import ctypes as C

import numpy as np
import pytest
import torch

import casegen as cg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


# one tile (no shared node); tiles of 16 elements (almost every node shared);
# the default; FP32 workgroups that walk several tiles
@pytest.mark.parametrize("tile_elems,cap", [(1024, 0), (16, 0), (0, 0), (64, 8)])
@pytest.mark.parametrize("op", [8, 1, 2, 4, 7])
def test_matches_internal_order(sw, tile_elems, cap, op):
    ctx = sw.Context(0)
    ctx.set_grid_cap(cap)
    mesh = cg.box_mesh(20.0, 20.0, 10.0, 5.0, jitter=0.2) if tile_elems == 1024 else cg.box_mesh(
        50.0, 40.0, 30.0, 5.0, jitter=0.2)
    case = cg.make_case(mesh, cg.CONFIGS["small"], n_steps=2, n_rec=2)
    gc = sw.Case(ctx, sw.Mesh(ctx, mesh, tile_elems=tile_elems), case, precision="mixed")
    n = 3 * mesh.n_nodes
    g = torch.Generator("cuda").manual_seed(op)
    x = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    for xd, call, eps in ((x, ctx.lib.sw_case_apply, 2.3e-16), (x.float(), ctx.lib.sw_case_apply_f32, 1.2e-7)):
        guard = torch.full((n + 16,), 7.0, dtype=xd.dtype, device="cuda")
        y = guard[8:n + 8]
        src = xd.clone()
        torch.cuda.synchronize()
        assert call(gc.h, op, C.c_void_p(src.data_ptr()), C.c_void_p(y.data_ptr())) == 0
        assert torch.equal(src, xd)
        assert bool((guard[:8] == 7.0).all()) and bool((guard[n + 8:] == 7.0).all())
        assert call(gc.h, op, C.c_void_p(src.data_ptr()), C.c_void_p(src.data_ptr())) == 0
        # the same arithmetic but for the order in which the up to 8 partial
        # sums of a tile and of a shared node's tiles (64 together) arrive
        assert float((src - y).abs().max()) <= 64 * eps * float(y.abs().max())
        # a second call finds the accumulators clear
        z = torch.empty_like(xd)
        torch.cuda.synchronize()
        assert call(gc.h, op, C.c_void_p(xd.data_ptr()), C.c_void_p(z.data_ptr())) == 0
        assert float((z - y).abs().max()) <= 64 * eps * float(y.abs().max())
