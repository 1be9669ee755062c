"""States whose ions lie so close together that the near / far split would cost
more than the direct sum take the direct sum, and only those; and the sorts of
the split and of the cutoff in bins that hold thousands of ions."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_06557_amd import workloads as W
from tests.gpu_util import accel_errors, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


def _ball(w, frac, rad, seed=5):
    """Uniform ions, `frac` of them in a ball of `rad` Debye lengths."""
    rng = np.random.default_rng(seed)
    n, R, H = w.n_ions, w.R / w.lam, w.H / w.lam
    r, p = R * np.sqrt(rng.uniform(size=n)), rng.uniform(0, 2 * np.pi, n)
    x = np.stack([r * np.cos(p), r * np.sin(p), H * (rng.uniform(size=n) - 0.5)])
    k = rng.permutation(n)[: int(n * frac)]
    d = rng.normal(size=(3, len(k)))
    x[:, k] = 0.9 + rad * d / np.linalg.norm(d, axis=0) * rng.uniform(size=len(k)) ** (1 / 3)
    return x.astype(np.float32)


def _accel(B, w, x, kind):
    with B.System(w) as s:
        s.set_pair_kernel(kind)
        s.set_state(x, np.zeros_like(x))
        s.step(1)
        s.sync()
        return s.accelerations()


# fractions and radii whose cost, by the measured 0.34 us per ion of the fullest
# column and 1.1 ps per near pair, is at least twice or at most two thirds of
# the direct sum's
@pytest.mark.parametrize("n_ions,frac,rad,direct", [
    (40960, 0.0, 1.0, False), (40960, 0.01, 0.1, False), (40960, 0.3, 0.1, True), (40960, 1.0, 0.05, True),
    (65537, 0.0, 1.0, False), (65537, 0.02, 0.1, False), (65537, 0.2, 0.1, True), (65537, 1.0, 1.0, True),
    (131072, 0.05, 0.1, False), (131072, 0.5, 0.1, True), (131072, 1.0, 0.02, True),
    (262145, 0.05, 0.1, False), (262145, 1.0, 0.1, True),
])
def test_route_of_dense_states(B, n_ions, frac, rad, direct):
    w = W.single_grain_small().with_(n_ions=n_ions, dust=[])
    x = _ball(w, frac, rad)
    a, d = _accel(B, w, x, B.PAIR_AUTO), _accel(B, w, x, B.PAIR_SYMMETRIC)
    assert np.array_equal(a, d) == direct
    if not direct:
        # the bounds of the direct FP32 sum, against the oracle: in such states, with their close
        # pairs, the direct kernel itself is 1.1e-6 off, from its terms' exponents
        o = O.Oracle(w, init=False)
        lam, wpi = o.derived["lam"], o.derived["wpi"]
        o.set_state(x.T.astype(np.float64) * lam, np.zeros((n_ions, 3)), np.zeros(0), 0)
        idx = np.random.default_rng(1).choice(n_ions, 1500, replace=False)
        l2, p999, _ = accel_errors(a.T.astype(np.float64)[idx], o.accel_subset(idx) / (lam * wpi * wpi))
        say("dense", n_ions, frac, rad, ":", l2, p999)
        assert l2 < 1e-6 and p999 < 3e-6


def test_dense_member_of_a_batch(B):
    ws = [W.single_grain_small().with_(n_ions=n, system_id=k, dust=[]) for k, n in enumerate((41001, 3000, 50003))]
    with B.Batch(ws) as b:
        b.step(1)
        for dense in (2, 0):
            xs = [_ball(w, 1.0 if k == dense else 0.0, 0.05) for k, w in enumerate(ws)]
            for k, x in enumerate(xs):
                b.set_state(k, x, np.zeros_like(x))
            b.step(1)
            b.sync()
            for k, w in enumerate(ws):
                kind = B.PAIR_SYMMETRIC if k == dense else B.PAIR_AUTO
                assert np.array_equal(b.accelerations(k), _accel(B, w, xs[k], kind)), (dense, k)


@pytest.mark.parametrize("n_ions,frac,rad", [(20000, 1.0, 0.02), (20000, 0.3, 0.1), (70001, 1.0, 0.1)])
def test_cutoff_sort_of_dense_states(B, n_ions, frac, rad):
    w = W.single_grain_small().with_(n_ions=n_ions, dust=[])
    x = _ball(w, frac, rad)
    o = O.Oracle(w, init=False)
    o.set_cutoff(1.0 * w.lam, 1.5 * w.lam)
    lam, wpi = o.derived["lam"], o.derived["wpi"]
    o.set_state(x.T.astype(np.float64) * lam, np.zeros((n_ions, 3)), np.zeros(0), 0)
    acc = []
    for _ in range(2):
        with B.System(w) as s:
            s.set_cutoff(1.0 * w.lam, 1.5 * w.lam)
            s.set_state(x, np.zeros_like(x))
            s.step(1)
            s.sync()
            acc.append(s.accelerations())
    assert np.array_equal(acc[0], acc[1])
    idx = np.random.default_rng(3).choice(n_ions, 400, replace=False)
    l2, p999, _ = accel_errors(acc[0].T.astype(np.float64)[idx], o.accel_subset(idx) / (lam * wpi * wpi))
    say("dense cutoff", n_ions, frac, rad, ":", l2, p999)
    assert l2 < 1e-6 and p999 < 3e-6
