"""CG iterations of two kernels (the direction formed inside the operator
pass) against the three-kernel iterations that the profiler asks for: the
same arithmetic up to the arrival order of the additions."""
import numpy as np
import pytest

import casegen as cg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


def _march(sw, mesh, case, three, steps, tiles, **kw):
    ctx = sw.Context(0)
    gm = sw.Mesh(ctx, mesh, tile_elems=tiles)
    gc = sw.Case(ctx, gm, case, **kw)
    gc.set_state(v=cg.smooth_field(mesh, 3, 30.0, 1e-2).ravel())
    ctx.profile(three)
    gc.step(steps)
    ctx.profile(False)
    return gc.waveforms(), gc.step_log()[0], gc.stats(), gm.info()[0]


# one tile; a few; more tiles than compute units; 1024-element tiles (several
# elements per work-item)
@pytest.mark.parametrize("tiles,box", [(1024, (10.0, 20.0, 20.0)), (64, (30.0, 40.0, 20.0)), (16, (50.0, 60.0, 40.0)),
                                       (1024, (60.0, 70.0, 50.0))])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "flex"])
def test_two_kernel_iterations_match_three(sw, tiles, box, precision):
    mesh = cg.box_mesh(*box, 5.0, jitter=0.2)
    case = cg.make_case(mesh, cg.CONFIGS["small"], n_steps=4, n_rec=2)
    kw = dict(precision=precision, guess="poly", rtol=1e-12)
    w2, it2, s2, nt = _march(sw, mesh, case, False, 4, tiles, **kw)
    w3, it3, s3, _ = _march(sw, mesh, case, True, 4, tiles, **kw)
    print(nt, it2, it3, np.linalg.norm(w2 - w3) / np.linalg.norm(w3))
    assert s2["flags"] == s3["flags"] == 0
    # a solve may stop one iteration apart where rounding decides (three rounds a step)
    assert np.all(np.abs(it2 - it3) <= 3)
    # both solve each step to 1e-12 of the right-hand side; the velocity error
    # of a step is that times the condition of the step operator (about 1e2)
    assert np.linalg.norm(w2 - w3) <= 1e-9 * np.linalg.norm(w3)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("max_iter", [1, 2, 7, 24])
def test_iteration_cap(sw, precision, max_iter):
    """The cap ends a solve after exactly max_iter iterations, inside a chunk,
    at its end and inside a replayed graph alike."""
    mesh = cg.box_mesh(30.0, 30.0, 20.0, 5.0)
    case = cg.make_case(mesh, cg.CONFIGS["small"], n_steps=2, n_rec=2)
    for three in (False, True):
        _, it, st, _ = _march(sw, mesh, case, three, 2, 64, precision=precision, guess="zero", rtol=1e-13,
                              max_iter=max_iter)
        assert list(it) == [max_iter, max_iter] and st["flags"] == 1, (it, st)
