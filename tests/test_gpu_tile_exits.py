"""The tile list builder's launch shapes and the two exits by which it leaves
a tile to the lane builder's walk: more particles around the tile than its LDS
slots, more steps than its step table.  The rules are followed here on the CPU
for every tile, so that each case is known to take the path it is named after;
rows are whole numbers and equal the oracle's brute-force rows."""
import math

import numpy as np
import pytest

import dpd_inputs as di
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_1311_0402_amd")

TILE = (8, 4, 4)
UNION = tuple(t + 2 for t in TILE)
CELLS = 128                       # of a tile
CAND = 4                          # slots of a step
KERNELS = (6, 7, 8, 10, 12, 16)   # waves of the instances


def _kernel_waves(n, n_cells):
    """Waves of the instance that n particles in n_cells cells get."""
    mean = CELLS * n / n_cells
    need = min(max(math.ceil((mean + 1.5 * math.sqrt(mean)) / 64), 6), 16)
    return next(k for k in KERNELS if need <= k)


def _capacity(waves):
    """LDS slots and steps of an instance."""
    slots = (waves * 64 * 29 // 10 + 15) // 16 * 16
    return slots, CELLS * ((slots * 27 // 360 + CAND - 1) // CAND + 8)


def _union_order():
    """The union cells in their order in LDS: by neighbouring tile, then Morton."""
    def key(c):
        k = 0
        for d in range(3):
            k = 3 * k + (0 if c[d] == 0 else 2 if c[d] == TILE[d] + 1 else 1)
        for b in range(3, -1, -1):
            for d in (2, 1, 0):
                k = 2 * k + ((c[d] + TILE[d] - 1) % TILE[d] >> b & 1)
        return k
    cells = [(x, y, z) for z in range(UNION[2]) for y in range(UNION[1]) for x in range(UNION[0])]
    return sorted(cells, key=key)


def _tile_loads(s):
    """(particles around it, steps of its cells) of every tile."""
    nc = [int(c) for c in oracle.cell_grid(s.box, s.r_c)]
    rank = np.asarray(oracle.morton_rank_table(nc)).reshape(nc[2], nc[1], nc[0])
    c = [np.minimum((s.x[d] * (nc[d] / s.box[d])).astype(int), nc[d] - 1) for d in range(3)]
    count = np.zeros_like(rank)
    np.add.at(count, (c[2], c[1], c[0]), 1)
    loads = []
    for oz in range(0, nc[2], TILE[2]):
        for oy in range(0, nc[1], TILE[1]):
            for ox in range(0, nc[0], TILE[0]):
                o = (ox, oy, oz)
                v = [min(TILE[d], nc[d] - o[d]) for d in range(3)]
                slots, at = {}, 0
                for u in _union_order():
                    if all(u[d] < v[d] + 2 for d in range(3)):
                        w = [(o[d] + u[d] - 1) % nc[d] for d in range(3)]
                        k = int(count[w[2], w[1], w[0]])
                        slots[u] = (int(rank[w[2], w[1], w[0]]), at, at + k)
                        at += k
                steps = 0
                for z in range(v[2]):
                    for y in range(v[1]):
                        for x in range(v[0]):
                            st = sorted(slots[x + i, y + j, z + k] for i in range(3) for j in range(3) for k in range(3))
                            runs = []
                            for _, a, b in st:
                                if a == b:
                                    continue
                                if runs and runs[-1][1] == a:
                                    runs[-1][1] = b
                                else:
                                    runs.append([a, b])
                            steps += 1 + sum(-(-(b - a) // CAND) for a, b in runs)
                loads.append((at, steps))
    return np.array(loads), nc[0] * nc[1] * nc[2]


def _assert_rows(s):
    sim = P.System(P.Params.like(s), s.n, P.FP64)
    sim.load(s.x, s.v, s.tag, s.type, step=0)
    torch.cuda.synchronize()
    x = sim.host_state()[0]
    off, idx = sim.host_nlist()
    off_ref, idx_ref = oracle.neighbors(x, s.box, s.r_c)
    np.testing.assert_array_equal(off, off_ref)
    np.testing.assert_array_equal(idx, idx_ref)
    return np.diff(off)


@pytest.mark.parametrize("waves", KERNELS)
def test_rows_of_every_instance(waves):
    """17 x 9 x 5 cells, so that tiles are clipped at every high face, at the
    density whose tiles need half a wave less than the instance has."""
    box = (17.3, 9.4, 5.2)
    lanes = 64.0 * (waves - 0.5)
    mean = (math.sqrt(lanes + 0.5625) - 0.75) ** 2
    s = di.uniform_fluid(int(mean * 17 * 9 * 5 / CELLS), box, 81)
    loads, n_cells = _tile_loads(s)
    assert n_cells == 17 * 9 * 5 and _kernel_waves(s.n, n_cells) == waves
    slots, steps = _capacity(waves)
    assert np.all(loads <= (slots, steps))
    _assert_rows(s)


def _full_tile(sites, seed):
    """Tile (1, 1, 1) alone filled, `sites` jittered lattice sites a cell, in a
    thin fluid; 25 x 13 x 13 cells."""
    box = np.array([25.3, 13.2, 13.2])
    side = box / (25, 13, 13)
    s = di.uniform_fluid(2200, box, seed)
    inside = np.all([(s.x[d] >= (TILE[d] - 1) * side[d]) & (s.x[d] < (2 * TILE[d] + 1) * side[d]) for d in range(3)],
                    axis=0)
    rng = np.random.default_rng(seed)
    grid = [np.arange(TILE[d] * sites[d]) / sites[d] + 0.5 / sites[d] + TILE[d] for d in range(3)]
    fill = np.stack([g.ravel() for g in np.meshgrid(*grid, indexing="ij")])
    fill = (fill + rng.uniform(-0.1, 0.1, fill.shape)) * side[:, None]
    t = di.uniform_fluid(int(np.count_nonzero(~inside)) + fill.shape[1], box, seed)
    t.x[:] = np.concatenate([s.x[:, ~inside], fill], axis=1)
    return t


def test_tile_with_more_steps_than_its_table():
    """1,024 particles, all in the tile's own cells, so that many stencils hold
    each: they fit the slots, their steps do not fit the table.  Rows fit the
    slab, and the walk of the tile left over writes them."""
    s = _full_tile((2, 2, 2), 82)
    loads, n_cells = _tile_loads(s)
    slots, steps = _capacity(_kernel_waves(s.n, n_cells))
    left = loads[:, 1] > steps
    assert np.count_nonzero(left) == 1 and np.all(loads[:, 0] <= slots)
    assert _assert_rows(s).max() <= 48


def test_tile_with_more_particles_than_its_slots():
    s = _full_tile((3, 3, 1), 83)
    loads, n_cells = _tile_loads(s)
    slots, _ = _capacity(_kernel_waves(s.n, n_cells))
    assert np.count_nonzero(loads[:, 0] > slots) == 1
    _assert_rows(s)


def test_more_steps_than_the_table_with_rows_over_the_slab():
    """A blob in a corner of its tile: the rows overflow the slab too, and the
    direct pass writes them at the offsets that the left tile's walk counted."""
    s = di.clustered_fluid(seed=14, box=(17.3, 9.4, 9.2), n_cluster=750, n_rest=900, size=2.0)
    s.x[:] = (s.x + np.array([3.0, 0.9, 0.9])[:, None]) % s.box[:, None]
    loads, n_cells = _tile_loads(s)
    slots, steps = _capacity(_kernel_waves(s.n, n_cells))
    assert np.any((loads[:, 0] <= slots) & (loads[:, 1] > steps))
    assert _assert_rows(s).max() > 48
