"""The cutoff sum's box classes (skipped, plain, switched) and its sort, where
they can go wrong: few ions, ragged tiles, cutoffs below the size of a box and
beyond the domain, narrow and wide switching intervals, ions outside the domain."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_06557_amd import workloads as W
from tests.gpu_util import accel_errors, say, to_oracle

pytestmark = pytest.mark.gpu
LAM = W.single_grain_small().lam

# FP32 pair terms of about ten roundings (3e-7 of a term), summed in FP32 over
# 256 ions at a time and in 64 bits beyond
L2, P999 = 1e-6, 3e-6


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


@pytest.mark.parametrize("n_ions,R,H,r_sw,r_cut", [
    (2, 3, 6, 1.0, 2.0),
    (257, 3, 6, 1.0, 2.0),
    (5001, 3, 6, 0.05, 0.1),        # below the size of a box: nearly all skipped
    (12345, 3, 12, 2.9, 3.0),       # narrow switch
    (12345, 3, 12, 0.0, 3.0),       # never plain
    (20011, 0.5, 40, 3.0, 4.0),     # thin: one cell across
    (20011, 9, 1.5, 1.5, 2.5),      # flat: one or two layers
    (16640, 3, 6, 20.0, 30.0),      # everything plain
])
def test_classes_match_oracle(B, n_ions, R, H, r_sw, r_cut):
    w = W.single_grain_small().with_(n_ions=n_ions, R=R * LAM, H=H * LAM, dust=[])
    o = O.Oracle(w, init=False)
    o.set_cutoff(r_sw * LAM, r_cut * LAM)
    with B.System(w) as s:
        s.set_cutoff(r_sw * LAM, r_cut * LAM)
        for outside in (False, True):
            if outside and n_ions > 100:
                x, v, q, n = s.get_state()
                x[:, :7] += (0.4 * np.array([R, R, H]))[:, None] * np.linspace(1.0, 3.0, 7)
                s.set_state(x, v, q, n)
            to_oracle(s, o)
            z = s.get_state()[0][2]
            s.step(1)
            s.sync()
            a = s.accelerations().T.astype(np.float64)
            lam, wpi = o.derived["lam"], o.derived["wpi"]
            idx = np.unique(np.concatenate([np.arange(min(n_ions, 40)), np.arange(max(n_ions - 40, 0), n_ions),
                                            np.random.default_rng(3).choice(n_ions, min(n_ions, 400), replace=False)]))
            l2, p999, _ = accel_errors(a[idx] * lam * wpi * wpi, o.accel_subset(idx))
            say("cutoff", n_ions, R, H, r_sw, r_cut, "outside" if outside else "", l2, p999)
            assert l2 < L2 and p999 < P999
            # the reported slabs and pairs are those of ions sorted by slab alone
            ns, pairs = s.cutoff_info()
            sl = np.clip(((z + np.float32(0.5 * H)) * np.float32(ns / H)).astype(np.int64), 0, ns - 1)
            sl.sort()
            reach = max(1, int(np.ceil(r_cut * ns / H)))
            hi = sl[np.minimum(np.arange(0, n_ions, 256) + 256, n_ions) - 1]
            je = np.searchsorted(sl, np.minimum(hi + reach + 1, ns))
            tiles = (je + 255) // 256 - np.arange(len(hi))
            assert abs(pairs - (65536 * (2 * tiles - 1)).sum()) <= 4 * 65536
