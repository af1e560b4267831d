"""FP64 forces of isolated pairs at the edges of the pair arithmetic: nearly
coincident, just inside and just outside r_c, across the periodic faces, and
every weight exponent (its own square root for s = 1/2).  1,000 pairs a
system draw 1,000 pair variates.

Tolerance per particle: 16 ulp (2^-53) of a + gamma |v_ij| + 7 sigma /
sqrt(dt), the largest sum the terms can reach (a variate stays below 6.8);
just inside r_c an ulp of r changes sqrt(w_C) by 2^-53 / (2 sqrt(1e-6)), 56
ulp of the noise term: 1e-12 of that sum covers both."""
import numpy as np
import pytest

import dpd_inputs as di
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_1311_0402_amd")

SEP = (1e-6, 0.01, 0.3, 0.7, 1.0 - 1e-6, 1.0 + 1e-9)


@pytest.mark.parametrize("s_exp", [0.5, 1.0, 2.0, 0.25])
def test_isolated_pairs(s_exp):
    rng = np.random.default_rng(61)
    m, side = 10, 30.0
    site = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij")).reshape(3, -1) * 3.0 + 0.05
    u = rng.normal(size=site.shape)
    u /= np.linalg.norm(u, axis=0)
    sep = np.resize(SEP, site.shape[1])
    x = np.concatenate([site, (site + u * sep) % side], axis=1)
    n = x.shape[1]
    s = di.uniform_fluid(n, (side,) * 3, 62, s=s_exp)
    s.x[:] = x
    sim = P.System(P.Params.like(s), n, P.FP64)
    sim.load(s.x, s.v, s.tag, s.type, step=0)
    sim.compute_forces(5)
    torch.cuda.synchronize()
    x, v, f, tag, typ = sim.host_state()
    f_ref, _, npair, _ = oracle.forces(s, x, v, tag, typ, 5, with_scale=True)
    order = np.argsort(tag)
    hit = np.sum(np.abs(f[:, order]), axis=0) > 0
    np.testing.assert_array_equal(hit, np.tile(sep < 1.0, 2))
    tol = 1e-12 * (25.0 + 4.5 * 2.0 * np.abs(v).max() * 3**0.5 + 7.0 * 3.0 / s.dt**0.5)
    assert np.abs(f - f_ref).max() <= tol
