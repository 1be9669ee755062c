"""The FP64 pair sum (each pair once, two-word totals) against the sum in
extended precision, at the edges of its tiles, work splits and number range."""
import numpy as np
import pytest

from paper_2205_06557_amd import workloads as W
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

# a term rounds about 20 times (10 of them in the square root and the
# exponential): 20 units of 1.1e-16, and r (up to 8) times the last place of the
# exponent's argument, 8 more; the sums add less than one
REL = 28 * 1.2e-16


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


def _bare(n):
    return W.single_grain_small().with_(n_ions=n, dust=[], mach=0.0, nu_in=0.0, E_ext=0.0)


def _exact(w, x, idx):
    L = np.longdouble
    X = x.astype(L)
    R, H = w.R / w.lam, w.H / w.lam
    out = np.zeros((3, len(idx)))
    for k, i in enumerate(idx):
        d = X[:, i:i + 1] - X
        r2 = (d * d).sum(axis=0)
        r2[i] = 1
        r = np.sqrt(r2)
        f = (1 + r) * np.exp(-r) / (r2 * r)
        f[i] = 0
        out[:, k] = ((f * d).sum(axis=1) * L(R * R * H / 4) / w.n_ions).astype(float)
    return out


def _errors(w, s, idx):
    x = s.get_state()[0]
    s.step(1)
    s.sync()
    a, r = s.accelerations()[:, idx], _exact(w, x, idx)
    return np.linalg.norm(a - r) / np.linalg.norm(r)


@pytest.mark.parametrize("n", [2, 65, 257, 3001, 8193, 20000, (1 << 16) + 600])
def test_sum_matches_extended_precision(B, n):
    w = _bare(n)
    idx = np.unique(np.concatenate([np.arange(min(n, 20)), np.arange(max(n - 20, 0), n),
                                    np.random.default_rng(n).choice(n, min(n, 60), replace=False)]))
    with B.System(w, precision=B.PREC_FP64) as s:
        for _ in range(2):
            e = _errors(w, s, idx)
            say("FP64 sum, N", n, "relative error", e)
            assert e < REL


def test_close_and_coincident_pairs(B):
    """A pair beyond the totals' range is summed one-sided, in that step only;
    coincident ions spoil their own accelerations and no others."""
    w = _bare(3001)
    with B.System(w, precision=B.PREC_FP64) as s, B.System(w, precision=B.PREC_FP64) as t:
        x0, v0, q0, n0 = s.get_state()
        x = x0.copy()
        x[:, 2000] = x[:, 7] + 1e-9
        s.set_state(x, np.zeros_like(v0), q0, n0)
        e = _errors(w, s, np.array([0, 7, 300, 2000, 3000]))
        say("close pair, relative error", e)
        assert e < REL
        s.set_state(x, np.zeros_like(v0), q0, n0)
        far = np.array([0, 300, 1999, 3000])        # unspoilt by the pair
        assert _errors(w, s, far) < 1e-14           # 3,000 terms added one by one
        for u in (s, t):                            # the same step number again, without the pair
            u.set_state(x0, v0, q0, n0)
            u.step(2)
        for a, b in zip(s.get_state()[:2], t.get_state()[:2]):
            assert np.array_equal(a, b)
        x[:, 2000] = x[:, 7]
        s.set_state(x, np.zeros_like(v0), q0, n0)
        s.step(1)                                   # 0 times infinity, for these two only
        bad = ~np.isfinite(s.accelerations()).all(axis=0)
        assert np.array_equal(np.nonzero(bad)[0], [7, 2000])
