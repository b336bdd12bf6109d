"""The trace summary of the tile kernels as they are: every instance of one
kernel by itself, and the busy time over the passes of the CG iterations."""
import sqlite3

from paper_2404_17754_amd import profsum


def _trace(tmp_path, rows):
    db = tmp_path / "trace.db"
    con = sqlite3.connect(db)
    con.execute("create table kernels (name text, start integer, end integer)")
    con.executemany("insert into kernels values (?, ?, ?)", rows)
    con.commit()
    con.close()
    out = tmp_path / "trace.txt"
    profsum.trace(str(db), str(out), "trace cmd")
    return out.read_text()


def test_capped_launches_do_not_set_the_bar(tmp_path):
    # the pass takes 320 and 330 us (one early exit); the autotuner's capped
    # candidates 430 and 670, of which 320 is less than half
    one = "void sw::k_tile<float, 256, 0, 1, false, false>(sw::MeshDev, unsigned char const*)"
    capped = "void sw::k_tile<float, 256, 0, 1, false, true>(sw::MeshDev, unsigned char const*)"
    txt = _trace(tmp_path, [(one, 0, 320_000), (one, 400_000, 730_000), (one, 800_000, 805_000),
                            (capped, 0, 430_000), (capped, 0, 670_000)])
    assert "k_tile<float, 256, 0, 1, false, false>: 3 launches" in txt
    assert "mean over 2 full launches 325.0 us" in txt
    assert "k_tile<float, 256, 0, 1, false, true>: 2 launches" in txt
    assert "mean over 2 full launches 550.0 us" in txt


def test_passes_of_every_path(tmp_path):
    cg = "void sw::k_tile_cg<float, __half, 512, 3, 4>(sw::MeshDev)"
    rows = [(cg, 0, 10_000), (cg, 20_000, 30_000), ("void sw::k_tile_dir<double, 256, 2>(sw::MeshDev)", 0, 40_000),
            ("void sw::k_tile_lanes_cg<256>(sw::TileLane<float> const*)", 0, 50_000),
            ("void sw::k_tile<double, 256, 0, 0, false, false>(sw::MeshDev)", 100_000, 160_000),
            ("void sw::k_tile_rhs<256, false>(sw::MeshDev)", 200_000, 270_000), ("sw::k_newmark(long)", 0, 5_000)]
    txt = _trace(tmp_path, rows)
    for label, n in (("k_tile_cg<float", 2), ("k_tile_dir<double", 1), ("k_tile_lanes_cg<", 1), ("k_tile<double", 1),
                     ("k_tile_rhs<", 1)):
        assert f"{label}: {n} launches" in txt
    # over 0 .. 30 us the other kernels run too; the passes made once a step
    # have no span of their own
    assert "device busy over the span of the k_tile_cg<float launches (0.0 ms): 100.0 %" in txt
    assert "span of the k_tile<double" not in txt and "span of the k_tile_rhs<" not in txt
