"""Pairs at the last FP64 distance below the cutoff: r^2 is the number before
r_c^2, so the pair is inside, while a root rounded up puts it on r_c itself,
where w_C = 0 and the backward pass's w_R / w_C is 0 / 0.

r_c = 1: the correctly rounded root is the number before 1, w_C = 2^-53; forces
and gradients agree with the oracle, the forces within 1e-12 of the largest sum
of their terms, the gradients (each a product of a few terms, of one pair)
within 1e-9.  Other r_c: whatever the rounding of r and 1 / r_c, both are
finite."""
from fractions import Fraction
import math

import numpy as np
import pytest

import dpd_inputs as di
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_1311_0402_amd")


def _edge_pair(r_c):
    """dx, dy with fma(dy, dy, dx * dx) the number before r_c^2."""
    want = math.nextafter(r_c * r_c, 0.0)
    dx = r_c
    for _ in range(64):
        dx = math.nextafter(dx, 0.0)
        left = want - dx * dx
        if left > 0.0:
            dy = math.sqrt(left)
            if float(Fraction(dx * dx) + Fraction(dy) * Fraction(dy)) == want:
                return dx, dy
    raise AssertionError(r_c)


def _planted(r_c, s_exp, seed):
    dx, dy = _edge_pair(r_c)
    s = di.uniform_fluid(2, (4.0 * r_c,) * 3, seed, r_c=r_c, s=s_exp)
    s.x[:] = 0.0
    s.x[0, 1], s.x[1, 1] = dx, dy
    return s


def _force_and_gradient(s, step):
    sim = P.System(P.Params.like(s), s.n, P.FP64)
    sim.load(s.x, s.v, s.tag, s.type, step=0)
    sim.compute_forces(step)
    g = np.random.default_rng(step).standard_normal(s.x.shape)
    out = [torch.empty((3, s.n), dtype=torch.float64, device="cuda") for _ in range(2)]
    out += [torch.empty(1, dtype=torch.float64, device="cuda") for _ in range(2)]
    P.dpd_forces_backward(sim.params, sim.state, sim.cells, sim.nlist, step, torch.as_tensor(g, device="cuda"),
                          *out, sim.ws)
    torch.cuda.synchronize()
    x, v, f, tag, typ = sim.host_state()
    assert sim.host_nlist()[0][-1] == 2                      # the pair is listed
    return (x, v, tag, typ), f, g, [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("s_exp", [0.5, 1.0, 2.0, 0.25])
def test_last_distance_below_the_cutoff(s_exp):
    s = _planted(1.0, s_exp, 71)
    (x, v, tag, typ), f, g, grads = _force_and_gradient(s, 9)
    f_ref, _, npair = oracle.forces(s, x, v, tag, typ, 9)
    assert npair.sum() == 2
    tol = 1e-12 * (25.0 + 4.5 * 2.0 * np.abs(v).max() * 3**0.5 + 7.0 * 3.0 / s.dt**0.5)
    assert np.abs(f - f_ref).max() <= tol
    for got, want in zip(grads, oracle.forces_vjp(s, x, v, tag, typ, 9, g)):
        np.testing.assert_allclose(got.reshape(want.shape), want, rtol=1e-9, atol=1e-9 * np.abs(want).max())


@pytest.mark.parametrize("s_exp", [0.5, 1.0, 2.0, 0.25])
@pytest.mark.parametrize("r_c", [0.7, 0.9, 1.1, 1.3, 1.7, 2.0, 2.4])
def test_last_distance_below_any_cutoff_is_finite(r_c, s_exp):
    _, f, _, grads = _force_and_gradient(_planted(r_c, s_exp, 72), 10)
    assert np.all(np.isfinite(f))
    for got in grads:
        assert np.all(np.isfinite(got))
