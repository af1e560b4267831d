"""Positions outside [0, L): a particle is binned into the nearest cell and
listed by its geometry from there, by the tile builder as by the lane
builder: the same rows bit for bit, and i in j's row if j is in i's."""
import numpy as np
import pytest

import dpd_inputs as di

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_1311_0402_amd")


def _rows(s, kind, precision):
    prev = P.set_list_builder(kind)
    try:
        sim = P.System(P.Params.like(s), s.n, precision)
        sim.load(s.x, s.v, s.tag, s.type, step=0)
        torch.cuda.synchronize()
    finally:
        P.set_list_builder(prev)
    return sim.host_state(), *sim.host_nlist()


@pytest.mark.parametrize("precision", [P.FP64, P.MIXED])
@pytest.mark.parametrize("box", [(17.3, 9.4, 5.2), (25.0, 13.0, 11.0), (3.4, 3.2, 3.9)])
def test_rows_of_positions_outside_the_box(box, precision):
    s = di.uniform_fluid(int(3.0 * np.prod(box)), box, 57)
    # a fourth of a slab's particles at a face moved out of the box together,
    # by a little and by several cells, so that they keep neighbours among
    # themselves and in the box
    out = np.zeros(s.n, dtype=bool)
    for d, (by, far) in enumerate([(0.2, 0.9), (0.01, 2.3), (0.6, 4.5)]):
        low = (s.x[d] < 0.5) & (s.tag % 4 == d)
        high = (s.x[d] > box[d] - 0.5) & (s.tag % 4 == 3)
        s.x[d, low] -= 0.5 + by
        s.x[d, high] += 0.5 + (far if d else by)
        out |= low | high
    (x, _, f, tag, _), off, idx = _rows(s, 0, precision)
    (x2, _, f2, tag2, _), off2, idx2 = _rows(s, 2, precision)
    np.testing.assert_array_equal(tag, tag2)
    np.testing.assert_array_equal(off, off2)
    np.testing.assert_array_equal(idx, idx2)
    np.testing.assert_array_equal(f, f2)
    rows = np.repeat(np.arange(s.n), np.diff(off))
    assert set(zip(rows.tolist(), idx.tolist())) == set(zip(idx.tolist(), rows.tolist()))
    of_out = np.diff(off)[out[tag]]
    assert np.count_nonzero(of_out) > of_out.size // 2
