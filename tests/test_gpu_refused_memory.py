"""Where an allocation is refused after creation, the call fails and the system
goes on as it was: no step runs without its pair sum."""
import numpy as np
import pytest

from paper_2205_06557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


class _Giver:
    """torch's memory until `most` is set; then no block larger than that."""

    def __init__(self, B):
        self.most, self._a = None, B.TorchAllocator()
        give = self._a._a
        self._hook = B.ALLOC_FN(lambda ctx, n: None if self.most is not None and n > self.most else give(ctx, n))
        self.struct = B.Allocator(self._hook, self._a._f, None)


def _make(B, monkeypatch, cls, what):
    giver = _Giver(B)
    monkeypatch.setattr(B, "TorchAllocator", lambda: giver)
    s = cls(what, torch_memory=True)
    monkeypatch.undo()
    return s, giver


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def test_system_keeps_its_pair_sum(B, monkeypatch):
    w = W.single_grain_small().with_(n_ions=50003)
    s, giver = _make(B, monkeypatch, B.System, w)
    with s, B.System(w) as ref:
        s.step(1)
        ref.step(1)
        giver.most = 0
        with pytest.raises(B.OdError):
            s.set_pair_kernel(B.PAIR_SYMMETRIC)
        # neither the split's memory, given back for it, nor the work items are to be had
        for _ in range(3):
            with pytest.raises(B.OdError):
                s.step(1)
        giver.most = None
        s.step(1)
        ref.step(1)
        s.sync()
        for p, q in zip(s.get_state()[:3], ref.get_state()[:3]):
            assert _rel(p.astype(np.float64), q.astype(np.float64)) < 1e-6
        assert _rel(s.accelerations().astype(np.float64), ref.accelerations().astype(np.float64)) < 3e-6


@pytest.mark.parametrize("change", ["items", "one_row", "autotune", "symmetric"])
def test_batch_keeps_its_pair_sums(B, monkeypatch, change):
    ws = [W.single_grain_small().with_(n_ions=n, system_id=k) for k, n in enumerate((3000, 30001, 50003))]
    b, giver = _make(B, monkeypatch, B.Batch, ws)
    with b, B.Batch(ws) as ref:
        b.step(1)
        ref.step(1)
        kind, cfg = b.pair_kernel(), b.sym_config()
        giver.most = 0
        with pytest.raises(B.OdError):
            if change == "items":
                b.set_sym_config(items_target=20000)
            elif change == "one_row":
                b.set_sym_config(one_row=True)
            elif change == "autotune":
                b.autotune(None)
            else:
                b.set_pair_kernel(B.PAIR_SYMMETRIC)
        assert b.pair_kernel() == kind and b.sym_config() == cfg
        if change == "autotune":                # its one-sided candidates asked for no memory
            giver.most = None
        b.step(2)
        ref.step(2)
        b.sync()
        for k in range(len(ws)):
            for p, q in zip(b.get_state(k)[:3], ref.get_state(k)[:3]):
                assert np.array_equal(p, q)
            assert np.array_equal(b.accelerations(k), ref.accelerations(k))
            assert np.array_equal(b.forces(k), ref.forces(k))


def test_batch_without_the_splits_memory(B, monkeypatch):
    ws = [W.single_grain_small().with_(n_ions=n, system_id=k) for k, n in enumerate((3000, 50003))]
    b, giver = _make(B, monkeypatch, B.Batch, ws)
    with b:
        b.step(1)
        state = [b.get_state(k) for k in range(2)]
        b.set_pair_kernel(B.PAIR_SYMMETRIC)
        b.step(1)
        ref = [b.accelerations(k) for k in range(2)]
        for k in range(2):
            b.set_state(k, *state[k])
        giver.most = 4 << 20                    # the work list, not the split's memory
        b.set_pair_kernel(B.PAIR_AUTO)
        b.step(1)
        b.sync()
        for k in range(2):
            assert np.array_equal(b.accelerations(k), ref[k])
