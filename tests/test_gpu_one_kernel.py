"""CG iterations of one kernel (both sums of an iteration from one operator
pass) and of two, against the three-kernel iterations that the profiler asks
for: the same iterates up to rounding."""
import numpy as np
import pytest

import casegen as cg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


def _march(sw, mesh, case, three, steps, tile_elems, **kw):
    ctx = sw.Context(0)
    gm = sw.Mesh(ctx, mesh, tile_elems=tile_elems)
    gc = sw.Case(ctx, gm, case, **kw)
    gc.set_state(v=cg.smooth_field(mesh, 3, 30.0, 1e-2).ravel())
    ctx.profile(three)
    gc.step(steps)
    ctx.profile(False)
    return gc.waveforms(), gc.step_log()[0], gc.stats(), gm.info()


# nodes per work-item 1, 2 and 3 of a 512-wide workgroup (tiles of 16, 256 and
# 1024 elements; 0: the default tiles), of a 256-wide one in FP64 past 256
# tiles (16, 64, 256, 512 elements); past 1800 (FP32) and 900 (FP64) tiles two
# kernels
@pytest.mark.parametrize("precision,tile_elems,box", [
    ("mixed", 16, (40.0, 40.0, 40.0)), ("mixed", 256, (60.0, 60.0, 50.0)), ("mixed", 1024, (60.0, 60.0, 50.0)),
    ("mixed", 0, (30.0, 30.0, 30.0)), ("flex", 256, (60.0, 60.0, 50.0)), ("mixed", 16, (100.0, 100.0, 80.0)),
    ("fp64", 16, (40.0, 40.0, 30.0)), ("fp64", 256, (60.0, 60.0, 50.0)), ("fp64", 1024, (60.0, 60.0, 50.0)),
    ("fp64", 0, (30.0, 30.0, 30.0)), ("fp64", 16, (60.0, 60.0, 50.0)), ("fp64", 64, (100.0, 100.0, 60.0)),
    ("fp64", 256, (140.0, 140.0, 100.0)), ("fp64", 512, (160.0, 160.0, 110.0)), ("fp64", 16, (100.0, 100.0, 40.0))])
def test_matches_three_kernels(sw, precision, tile_elems, box):
    mesh = cg.box_mesh(*box, 5.0, jitter=0.2)
    case = cg.make_case(mesh, cg.CONFIGS["small"], n_steps=3, n_rec=2)
    kw = dict(precision=precision, guess="poly", rtol=1e-12)
    w1, it1, s1, info = _march(sw, mesh, case, False, 3, tile_elems, **kw)
    w3, it3, s3, _ = _march(sw, mesh, case, True, 3, tile_elems, **kw)
    print(info, it1, it3, np.linalg.norm(w1 - w3) / np.linalg.norm(w3))
    assert s1["flags"] == s3["flags"] == 0
    # rounding decides where a solve stops (one iteration a round) and, near the
    # tolerance, whether a last short round follows, which halves the residual
    # and so costs at least ln 2 / ln 1e12 of the step's 250 iterations, and a
    # restarted CG's first few: the three-kernel iterations alone give 237 and
    # 246 on one mesh with different tiles
    assert np.all(np.abs(it1 - it3) <= (3 if precision == "fp64" else 12))
    # both solve each step to 1e-12 of the right-hand side; the velocity error
    # of a step is that times the condition of the step operator (about 1e2)
    assert np.linalg.norm(w1 - w3) <= 1e-9 * np.linalg.norm(w3)


# 96 tiles of 64 to 384 elements, then 256 tiles, then 512 elements
@pytest.mark.parametrize("box,n_tets,tiles", [((20.0, 20.0, 20.0), 384, 6), ((100.0, 100.0, 50.0), 24000, 96),
                                              ((110.0, 110.0, 100.0), 58080, 152), ((160.0, 160.0, 80.0), 98304, 256),
                                              ((160.0, 160.0, 105.0), 129024, 256),
                                              ((200.0, 200.0, 70.0), 134400, 263)])
def test_default_tiles(sw, box, n_tets, tiles):
    mesh = cg.box_mesh(*box, 5.0)
    assert mesh.n_tets == n_tets
    assert sw.Mesh(sw.Context(0), mesh).info()[0] == tiles
