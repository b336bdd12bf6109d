"""CG iterations of two kernels where cases do run them: in FP64 past 900 tiles,
with FP32 inner solves from 1801 to 4000.  Against the three-kernel iterations
that the profiler asks for, which path ran asserted on both sides."""
import functools

import numpy as np
import pytest

import casegen as cg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


@functools.lru_cache(maxsize=1)
def _mesh(box):
    m = cg.box_mesh(*box, 5.0, jitter=0.2)
    return m, cg.make_case(m, cg.CONFIGS["small"], n_steps=3, n_rec=2), cg.smooth_field(m, 3, 30.0, 1e-2).ravel()


def _march(sw, box, three, steps, tile_elems, **kw):
    mesh, case, v = _mesh(box)
    ctx = sw.Context(0)
    gm = sw.Mesh(ctx, mesh, tile_elems=tile_elems)
    gc = sw.Case(ctx, gm, case, **kw)
    gc.set_state(v=v)
    ctx.profile(three)
    assert gc.schedule() == ((3, 0) if three else (2, 0))
    gc.step(steps)
    ctx.profile(False)
    return gc.waveforms(), gc.step_log()[0], gc.stats(), gm.info()[0]


# tiles of 16 elements; of up to 300 and of 512 (two elements and up to five
# nodes per FP64 work-item, three per FP32 one); the last box has more than 1.5
# million nodes, past which the vector kernel takes them as one stream
@pytest.mark.parametrize("precision,tile_elems,box", [
    ("fp64", 16, (100.0, 100.0, 40.0)), ("fp64", 300, (220.0, 220.0, 120.0)), ("fp64", 0, (270.0, 270.0, 135.0)),
    ("mixed", 16, (100.0, 100.0, 80.0)), ("flex", 16, (100.0, 100.0, 80.0)), ("mixed", 0, (380.0, 380.0, 140.0)),
    ("flex", 0, (380.0, 380.0, 140.0)), ("mixed", 0, (390.0, 390.0, 155.0)), ("fp64", 0, (390.0, 390.0, 155.0))])
def test_matches_three_kernels(sw, precision, tile_elems, box):
    kw = dict(precision=precision, guess="poly", rtol=1e-12)
    w2, it2, s2, tiles = _march(sw, box, False, 2, tile_elems, **kw)
    w3, it3, s3, _ = _march(sw, box, True, 2, tile_elems, **kw)
    print(tiles, it2, it3, np.linalg.norm(w2 - w3) / np.linalg.norm(w3))
    assert s2["flags"] == s3["flags"] == 0
    # rounding decides where a solve stops (one iteration a round) and, near the
    # tolerance, whether a last short mixed round follows
    assert np.all(np.abs(it2 - it3) <= (3 if precision == "fp64" else 12))
    # both solve each step to 1e-12 of the right-hand side; the velocity error
    # of a step is that times the condition of the step operator (about 1e2)
    assert np.linalg.norm(w2 - w3) <= 1e-9 * np.linalg.norm(w3)


@pytest.mark.parametrize("precision,box", [("fp64", (100.0, 100.0, 40.0)), ("mixed", (100.0, 100.0, 80.0)),
                                           ("flex", (100.0, 100.0, 80.0))])
@pytest.mark.parametrize("max_iter", [1, 2, 7, 10, 24])
def test_iteration_cap(sw, precision, box, max_iter):
    """The cap ends a solve after exactly max_iter iterations, inside a chunk,
    at its end and inside a replayed graph of eight."""
    for three in (False, True):
        _, it, st, _ = _march(sw, box, three, 2, 16, precision=precision, guess="zero", rtol=1e-13, max_iter=max_iter)
        assert list(it) == [max_iter, max_iter] and st["flags"] == 1, (it, st)


def test_graphs_and_direct_launches(sw):
    """Replayed graphs and direct launches of the same kernels, in FP64 and FP32."""
    for precision, box in (("fp64", (100.0, 100.0, 40.0)), ("mixed", (100.0, 100.0, 80.0))):
        mesh, case, v = _mesh(box)
        w = []
        for graphs in (True, False):
            ctx = sw.Context(0)
            ctx.set_graphs(graphs)
            gc = sw.Case(ctx, sw.Mesh(ctx, mesh, tile_elems=16), case, precision=precision, guess="poly", rtol=1e-12)
            gc.set_state(v=v)
            assert gc.schedule() == (2, 0)
            gc.step(3)
            w.append(gc.waveforms())
            assert gc.stats()["flags"] == 0
        assert np.linalg.norm(w[0] - w[1]) <= 1e-9 * np.linalg.norm(w[1])
