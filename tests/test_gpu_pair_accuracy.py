"""Errors of the FP64 pair arithmetic against 64-bit-mantissa references
(numpy long double): the variate, over words that a sweep draws and over edge
words planted through the inverse of Philox, and distances and directions, from
conservative forces of single pairs.

Bounds are sums of the steps' errors in units of 2^-53 relative: a rounding 1,
the logarithm 3 (its result's, its inner sum's and s's rounding), a root 1 and
half its argument's, the cosine 3 (an ulp beside the rounded value), the
reciprocal distance 2, the squared distance 3.  A variate is a root of a
logarithm times a cosine: 1.5 + 1 + 3 + 1 = 6.5; as a force, times e = d / r
(2 + 1 for an exact r) and a product: 10.5.  A conservative force at r <= 1/2:
r 1.5 + 2, hence 3.5 in 1 - r and 1 for that difference, e 1.5 + 2 + 1, two
products: 11."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_1311_0402_amd")
from paper_1311_0402_amd import dpd as D  # noqa: E402

U = 2.0 ** -53
LD = np.longdouble
PI_LD = 4 * np.arctan(LD(1))
M0, M1, W0, W1 = 0xD2511F53, 0xCD9E8D57, 0x9E3779B9, 0xBB67AE85
M32 = 0xFFFFFFFF


def _variate(w0, w1):
    """sqrt(-2 ln u1) cos(2 pi u2) of the words, in long double; the quarter
    turns are taken off in integers."""
    w0, w1 = np.asarray(w0, dtype=np.uint64), np.asarray(w1, dtype=np.int64)
    u1 = (w0.astype(LD) + LD(0.5)) * LD(2.0) ** -32
    q = (w1 + (1 << 29)) >> 30
    x = (w1 - (q << 30)).astype(LD) * LD(2.0) ** -30 * PI_LD / 2
    q = q % 4
    turn = np.where(q % 2 == 0, np.cos(x), np.sin(x)) * np.where((q == 1) | (q == 2), -1, 1)
    return np.sqrt(-2 * np.log(u1)) * turn


def _rel(got, want):
    zero = want == 0
    assert np.all(np.asarray(got)[zero] == 0)
    return np.abs((got[~zero].astype(LD) - want[~zero]) / want[~zero]).astype(np.float64)


def _unphilox(words, key):
    """The counter that Philox4x32-10 turns into these words."""
    c = list(words)
    i0, i1 = pow(M0, -1, 1 << 32), pow(M1, -1, 1 << 32)
    for r in range(9, -1, -1):
        k0, k1 = (key[0] + r * W0) & M32, (key[1] + r * W1) & M32
        x2, x0 = c[1] * i1 & M32, c[3] * i0 & M32
        c = [x0, c[0] ^ (x2 * M1 >> 32) ^ k0, x2, c[2] ^ (x0 * M0 >> 32) ^ k1]
    return c


def test_drawn_variates():
    n, step, seed = 1 << 20, (3 << 32) + 17, 0x123456789ABCDEF1
    sink = torch.empty(n, dtype=torch.float64, device="cuda")
    D.gaussian_throughput(0, n, 1, step, seed, None, sink)
    a = np.arange(n, dtype=np.uint64)
    b = (a + 1) % n
    c = [np.minimum(a, b), np.maximum(a, b), np.full(n, step & M32, np.uint64), np.full(n, step >> 32, np.uint64)]
    for r in range(10):
        k0, k1 = (seed + r * W0) & M32, ((seed >> 32) + r * W1) & M32
        p0, p1 = c[0] * np.uint64(M0), c[2] * np.uint64(M1)
        s32, m = np.uint64(32), np.uint64(M32)
        c = [(p1 >> s32) ^ c[1] ^ np.uint64(k0), p1 & m, (p0 >> s32) ^ c[3] ^ np.uint64(k1), p0 & m]
    rel = _rel(sink.cpu().numpy(), _variate(c[0], c[1]))
    print(f"variate: max {rel.max() / U:.2f}, rms {np.sqrt(np.mean(rel ** 2)) / U:.2f} (2^-53)")
    assert rel.max() <= 6.5 * U


@pytest.mark.parametrize("s_exp,r", [(1.0, 0.5), (0.5, 0.75)])
def test_planted_words(s_exp, r):
    """Forces of one pair whose only term is the random one, with sigma w_R =
    1: the variate itself."""
    seed = 0x0F1E2D3C4B5A6978
    key = (seed & M32, seed >> 32)
    half_root = int(2 ** 31.5)                     # u1 around sqrt(1/2): the logarithm's two branches
    w0 = [0, 1, 2, 3, 255, 1 << 16, 1 << 31, (1 << 31) - 1, half_root >> 1, half_root - 1, half_root, half_root + 1,
          half_root + 2, M32 - (1 << 20), M32 - 2, M32 - 1, M32]
    quarter = 1 << 30
    w1 = sorted({(k * (quarter >> 1) + d) & M32 for k in range(9) for d in (-2, -1, 0, 1, 2)})
    par = P.Params(box=(4.0, 4.0, 4.0), dt=1.0, s=s_exp, a=np.zeros((1, 1)), gamma=np.zeros((1, 1)),
                   sigma=np.full((1, 1), 2.0), seed=seed)
    sim = P.System(par, 2, P.FP64)
    x = np.zeros((3, 2))
    x[0, 1] = r
    sim.load(x, np.zeros((3, 2)), np.arange(2), np.zeros(2), step=0)
    at = int(sim.host_state()[0][0].argmax())      # the particle at +r: e = (1, 0, 0)
    rng = np.random.default_rng(91)
    words, forces = [], []
    for u in w0:
        for v in w1:
            while True:
                c = _unphilox((u, v, int(rng.integers(1 << 32)), int(rng.integers(1 << 32))), key)
                if c[0] < c[1]:
                    break
            sim.state.tag.copy_(torch.tensor(np.array(c[:2], dtype=np.uint32).view(np.int32)))
            sim.compute_forces(c[2] | c[3] << 32)
            words.append((u, v))
            forces.append(sim.state.f[0, at].clone())
    np.testing.assert_array_equal(oracle.philox(np.array([c], dtype=np.uint32), np.array([key], dtype=np.uint32))
                                  .ravel()[:2], words[-1])
    words = np.array(words, dtype=np.uint64)
    rel = _rel(torch.stack(forces).cpu().numpy(), _variate(words[:, 0], words[:, 1]))
    print(f"planted, s = {s_exp}: max {rel.max() / U:.2f} (2^-53)")
    assert rel.max() <= 10.5 * U


def test_conservative_forces_of_single_pairs():
    """2,000 systems of two particles, one at the origin, r from 1e-140 to 1/2."""
    n, rng = 2000, np.random.default_rng(92)
    r = np.concatenate([rng.uniform(0.0, 0.5, n // 2), np.exp(rng.uniform(np.log(1e-140), np.log(0.5), n // 2))])
    d = np.abs(rng.standard_normal((3, n)))
    d *= r / np.linalg.norm(d, axis=0)
    d[:, ::5] *= np.array([1.0, 0.0, 0.0])[:, None]
    par = [P.Params(box=(3.5, 3.3, 3.1), a=np.full((1, 1), 25.0), gamma=np.zeros((1, 1)), sigma=np.zeros((1, 1)), seed=k)
           for k in range(n)]
    sim = P.Batch(par, [2] * n, P.FP64)
    src = P.State.empty(2 * n)
    x = np.zeros((3, 2 * n))
    x[:, 1::2] = d
    src.x.copy_(torch.as_tensor(x))
    src.v.zero_()
    src.tag.copy_(torch.arange(2, dtype=torch.int32).repeat(n))
    src.type.zero_()
    sim.reorder_from(src)
    sim.rebuild()
    sim.compute_forces(0)
    st = sim.state
    f = st.f.cpu().numpy()[:, st.tag.cpu().numpy() == 1]
    dl = d.astype(LD)
    rl = np.sqrt(np.sum(dl * dl, axis=0))
    want = 25 * (1 - rl) * dl / rl
    rel = _rel(f, want)
    print(f"conservative: max {rel.max() / U:.2f} (2^-53)")
    assert rel.max() <= 11 * U
