"""The tile list builder (one workgroup per 8 x 4 x 4 cells) at the edges of
its launch shapes: workgroups of 6 to 16 waves (by density), tiles clipped at
the high faces, rows with more hits than a lane keeps before it writes them
out, and positions that are no numbers.  Rows are whole numbers: they equal
the oracle's brute-force rows, or the lane builder's, bit for bit."""
import numpy as np
import pytest

import dpd_inputs as di
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_1311_0402_amd")

BOX = (17.3, 9.4, 5.2)          # 17 x 9 x 5 cells: tiles of 8, 8, 1 x 4, 4, 1 x 4, 1


def _rows(s, kind=0):
    prev = P.set_list_builder(kind)
    try:
        sim = P.System(P.Params.like(s), s.n, P.FP64)
        sim.load(s.x, s.v, s.tag, s.type, step=0)
        torch.cuda.synchronize()
        x = sim.host_state()[0]
        off, idx = sim.host_nlist()
    finally:
        P.set_list_builder(prev)
    return x, off, idx


@pytest.mark.parametrize("density", [0.5, 3.0, 3.7, 4.6, 5.6, 7.0])     # 6, 7, 8, 10, 12, 16 waves
def test_rows_at_every_workgroup_size(density):
    n = int(density * BOX[0] * BOX[1] * BOX[2])
    s = di.uniform_fluid(n, BOX, 51)
    x, off, idx = _rows(s)
    off_ref, idx_ref = oracle.neighbors(x, s.box, s.r_c)
    np.testing.assert_array_equal(off, off_ref)
    np.testing.assert_array_equal(idx, idx_ref)


def test_rows_of_many_dense_tiles():
    """Beyond 512 tiles of 16 waves two workgroups share a compute unit: a
    seeded sample of 400 rows."""
    s = di.uniform_fluid(510_000, (74.3, 40.4, 24.2), 54)
    x, off, idx = _rows(s)
    q = np.sort(np.random.default_rng(54).choice(s.n, 400, replace=False)).astype(np.int32)
    off_ref, idx_ref = oracle.neighbors(x, s.box, s.r_c, query=q)
    for k, i in enumerate(q):
        np.testing.assert_array_equal(idx[off[i]:off[i + 1]], idx_ref[off_ref[k]:off_ref[k + 1]], err_msg=f"row {i}")


def test_rows_beyond_a_lanes_words():
    """A blob of density 10 in a fluid of density 3: rows of ~40 entries in
    the slab's 48, from more steps with a hit than a lane keeps words."""
    s = di.clustered_fluid(seed=52, box=(17.3, 9.4, 9.2), n_cluster=90, n_rest=4400, size=2.1)
    x, off, idx = _rows(s)
    off_ref, idx_ref = oracle.neighbors(x, s.box, s.r_c)
    assert np.diff(off).max() > 30
    np.testing.assert_array_equal(off, off_ref)
    np.testing.assert_array_equal(idx, idx_ref)


def test_positions_that_are_no_numbers_have_no_neighbours():
    s = di.uniform_fluid(1500, BOX, 53)
    bad = np.array([3, 4, 500, 501, 1499])
    s.x[0, bad[:3]] = np.nan
    s.x[2, bad[2:]] = np.nan
    _, off, idx = _rows(s)
    _, off_ref, idx_ref = _rows(s, kind=2)
    np.testing.assert_array_equal(off, off_ref)
    np.testing.assert_array_equal(idx, idx_ref)
    assert np.count_nonzero(np.diff(off) == 0) >= bad.size


@pytest.mark.parametrize("n", [1, 4095, 4096, 1024 * 4096 - 1, 1024 * 4096])
def test_offsets_at_the_scans_edges(n):
    """The scan of the n + 1 row sizes in one launch (to 4,096 items), in two
    (to 1,024 workgroups' 4,096 items) and in three: offsets of a seeded sample
    of rows, and their number, against the oracle's rows and the row lengths."""
    side = max(3.3, (n / 3.0) ** (1.0 / 3.0))
    s = di.uniform_fluid(n, (side,) * 3, 55)
    x, off, idx = _rows(s)
    assert off[0] == 0 and off[-1] == len(idx) and np.all(np.diff(off) >= 0)
    q = np.unique(np.concatenate([np.random.default_rng(55).choice(n, min(n, 60), replace=False), [0, n - 1]]))
    off_ref, idx_ref = oracle.neighbors(x, s.box, s.r_c, query=q.astype(np.int32))
    for k, i in enumerate(q):
        np.testing.assert_array_equal(idx[off[i]:off[i + 1]], idx_ref[off_ref[k]:off_ref[k + 1]], err_msg=f"row {i}")
    # every offset: rows ascend, so the list falls at row ends only
    down = np.nonzero(np.diff(idx) <= 0)[0] + 1
    assert np.all(np.isin(down, off))
