"""The near / far split of the all-pairs sum (large FP32 systems) against the
oracle's 64-bit direct sum and against the direct kernel, at the sizes, domain
shapes and ion distributions where it can go wrong."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_06557_amd import workloads as W
from tests.gpu_util import accel_errors, say

pytestmark = pytest.mark.gpu
LAM = W.single_grain_small().lam

# FP32 pair terms (1e-7 each, summed in 64 bits) and a far part within 1e-7 of
# the rms acceleration: the bounds of the direct FP32 sum at these sizes
L2, P999 = 1e-6, 3e-6


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


def _against_oracle(s, w, nt=1500):
    """One step; sampled accelerations against the oracle at the same state."""
    o = O.Oracle(w, init=False)
    x, v, q, step = s.get_state()
    lam, cs, wpi = o.derived["lam"], o.derived["cs"], o.derived["wpi"]
    o.set_state(x.T.astype(np.float64) * lam, v.T.astype(np.float64) * cs, q, step)
    s.step(1)
    s.sync()
    a = s.accelerations().T.astype(np.float64)
    idx = np.sort(np.random.default_rng(1).choice(w.n_ions, nt, replace=False))
    ref = o.accel_subset(idx) / (lam * wpi * wpi)
    return accel_errors(a[idx], ref)


@pytest.mark.parametrize("n_ions,R,H,grains", [
    (40960, 3, 6, 1),              # the smallest split system
    (81920, 3, 6, 1),
    ((1 << 17) + 1, 3, 6, 1),
    (100003, 1.5, 14, 1),          # long and thin
    (100003, 8, 2.5, 1),           # flat
    (200001, 3, 8, 8),             # chain of eight grains
    ((1 << 19) + 333, 3, 6, 1),    # another search schedule (four waves per tile)
])
def test_split_matches_oracle(B, n_ions, R, H, grains):
    w = W.chain8() if grains == 8 else W.single_grain_small()
    w = w.with_(n_ions=n_ions, R=R * LAM, H=H * LAM)
    with B.System(w) as s:
        l2, p999, top = _against_oracle(s, w)
        say("split, N", n_ions, "R", R, "H", H, ":", l2, p999, top)
        assert l2 < L2 and p999 < P999
        s.step(3)                  # after pushes and reinjections
        l2, p999, top = _against_oracle(s, w)
        assert l2 < L2 and p999 < P999


def _states(w, n):
    rng = np.random.default_rng(5)
    R, H = w.R / w.lam, w.H / w.lam
    uni = np.stack([R * np.sqrt(rng.uniform(size=n)), rng.uniform(0, 2 * np.pi, n), H * (rng.uniform(size=n) - 0.5)])
    uni = np.stack([uni[0] * np.cos(uni[1]), uni[0] * np.sin(uni[1]), uni[2]])
    dense = uni.copy()             # a third of the ions in a ball of a tenth of a Debye length
    k = n // 3
    d = rng.normal(size=(3, k))
    dense[:, :k] = 0.9 + 0.1 * d / np.linalg.norm(d, axis=0) * rng.uniform(size=k) ** (1 / 3)
    wall = uni.copy()              # on the side and on the end faces
    ph = rng.uniform(0, 2 * np.pi, n // 4)
    wall[0, : n // 4], wall[1, : n // 4] = R * np.cos(ph), R * np.sin(ph)
    wall[2, n // 4: n // 2] = 0.5 * H * np.sign(wall[2, n // 4: n // 2])
    out = uni.copy()               # some far outside the domain: this step is summed directly
    out[:, :5] = 40.0 + rng.uniform(size=(3, 5))
    return dict(dense=dense, wall=wall, outside=out)


@pytest.mark.parametrize("kind", ["dense", "wall", "outside"])
def test_split_of_unusual_states(B, kind):
    w = W.single_grain_small().with_(n_ions=82001, dust=[])
    with B.System(w) as s:
        s.set_state(_states(w, w.n_ions)[kind].astype(np.float32), np.zeros((3, w.n_ions), np.float32))
        l2, p999, top = _against_oracle(s, w)
        say("split, state", kind, ":", l2, p999, top)
        assert l2 < L2 and p999 < P999


def test_split_close_to_direct_and_reproducible(B):
    w = W.two_grain_wake().with_(n_ions=90001)
    runs = []
    for kind in (B.PAIR_AUTO, B.PAIR_AUTO, B.PAIR_SYMMETRIC):
        with B.System(w) as s:
            s.set_pair_kernel(B.PAIR_SYMMETRIC)
            s.set_pair_kernel(kind)
            s.step(1)
            a = s.accelerations()
            s.step(4)
            x, v, q, _ = s.get_state()
            runs.append((a, x, v, q, s.forces(0)))
    for p, q in zip(runs[0], runs[1]):
        assert np.array_equal(p, q)
    assert not np.array_equal(runs[0][0], runs[2][0])       # the split was in use
    l2, p999, _ = accel_errors(runs[0][0].T.astype(np.float64), runs[2][0].T.astype(np.float64))
    assert l2 < L2 and p999 < P999


def test_split_graph_replay_bitwise(B):
    import torch
    w = W.single_grain_small().with_(n_ions=82001)
    stream = torch.cuda.Stream()
    with B.System(w, stream=stream.cuda_stream) as g, B.System(w, stream=stream.cuda_stream) as e:
        g.set_graph(3)
        for k in (6, 4, 3):
            g.step(k)
            e.step(k)
            torch.zeros(1000, device="cuda").sum().item()       # other work between the replays
            for p, q in zip(g.get_state()[:3], e.get_state()[:3]):
                assert np.array_equal(p, q)


def test_split_reports_coincident_ions(B):
    w = W.single_grain_small().with_(n_ions=82000, dust=[])
    with B.System(w) as s:
        x = _states(w, w.n_ions)["wall"].astype(np.float32)
        x[:, 7] = x[:, 40000]
        s.set_state(x, np.zeros_like(x))
        s.step(1)
        with pytest.raises(B.OdError):
            s.sync()


def _members():
    c = W.chain8()
    base = [W.single_grain_small(), W.two_grain_wake(), c, c.with_(mach=0.6)]
    sizes = [3001, 41000, 65537, 50003]
    return [w.with_(n_ions=n, system_id=k) for k, (w, n) in enumerate(zip(base, sizes))]


@pytest.mark.parametrize("graph", [0, 2])
def test_split_batch_members_equal_single_runs(B, graph):
    """Members of a batch are split as they are when run alone, on whatever
    stream and scratch they fall; one state has ions outside the domain."""
    ws = _members()
    with B.Batch(ws) as b:
        if graph:
            b.set_graph(graph)
        b.step(3)
        x, v, q, n = b.get_state(2)
        out = x.copy()
        out[:, :3] = 30.0 + np.arange(3)
        b.set_state(2, out, v, q, n)
        b.step(4)
        b.sync()
        for k, w in enumerate(ws):
            with B.System(w) as s:
                s.step(3)
                if k == 2:
                    for p, r in zip(s.get_state()[:3], (x, v, q)):
                        assert np.array_equal(p, r)
                    s.set_state(out, v, q, n)
                s.step(4)
                for p, r in zip(b.get_state(k)[:3], s.get_state()[:3]):
                    assert np.array_equal(p, r), (k, w.n_ions)
                assert np.array_equal(b.accelerations(k), s.accelerations())
        b.set_pair_kernel(B.PAIR_SYMMETRIC)
        b.step(1)
        b.set_pair_kernel(B.PAIR_AUTO)
        b.step(1)
        b.sync()
