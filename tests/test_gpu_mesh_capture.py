"""A step of the near / far split whose ions lie outside the domain is summed
directly, also where the caller captured the step itself: before or after
od_set_state put the ions there."""
import numpy as np
import pytest

from paper_2205_06557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


def _outside(x, w):
    """Three ions beyond the side, three beyond an end face, one far away."""
    out = x.copy()
    R, H = w.R / w.lam, w.H / w.lam
    out[0, :3] = 1.01 * R + 0.1 * np.arange(3)
    out[2, 3:6] = -0.51 * H - 0.1 * np.arange(3)
    out[:, 6] = 40.0
    return out


def _after(B, w, state, kind, steps=3):
    """State and accelerations after one step and `steps` more, directly."""
    with B.System(w) as s:
        s.set_pair_kernel(kind)
        s.step(1)
        s.set_state(*state)
        s.step(1)
        a = s.accelerations()
        s.set_pair_kernel(B.PAIR_AUTO)
        s.step(steps)
        return a, s.get_state()


@pytest.mark.parametrize("n_ions", [40960, 65537])
@pytest.mark.parametrize("marked_first", [False, True])
def test_captured_step_after_set_state(B, n_ions, marked_first):
    import torch
    w = W.single_grain_small().with_(n_ions=n_ions)
    stream = torch.cuda.Stream()
    with B.System(w, stream=stream.cuda_stream) as s:
        s.step(2)
        inside = s.get_state()
        out = (_outside(inside[0], w),) + inside[1:]
        ref_a, ref = _after(B, w, out, B.PAIR_SYMMETRIC)
        if marked_first:                        # captured while the state has ions outside
            s.set_state(*out)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            s.step(1)
        for _ in range(2):                      # as often as the caller likes, either way round
            s.set_state(*out)
            with torch.cuda.stream(stream):
                g.replay()
            assert np.array_equal(s.accelerations(), ref_a)
            with torch.cuda.stream(stream):
                for _ in range(3):
                    g.replay()
            for p, q in zip(s.get_state()[:3], ref[:3]):
                assert np.array_equal(p, q)
            s.set_state(*inside)
            with torch.cuda.stream(stream):
                g.replay()
            with B.System(w) as e:
                e.set_state(*inside)
                e.step(1)
                assert np.array_equal(s.accelerations(), e.accelerations())
                assert not np.array_equal(s.accelerations(), ref_a)


def test_captured_batch_step_after_set_state(B):
    import torch
    c = W.chain8()
    ws = [c.with_(n_ions=n, system_id=k) for k, n in enumerate((3001, 41000, 50003))]
    stream = torch.cuda.Stream()
    with B.Batch(ws, stream=stream.cuda_stream) as b:
        b.step(2)
        x, v, q, n = b.get_state(2)
        out = (_outside(x, ws[2]), v, q, n)
        ref_a, ref = _after(B, ws[2], out, B.PAIR_SYMMETRIC)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            b.step(1)
        for _ in range(2):
            b.set_state(2, *out)
            with torch.cuda.stream(stream):
                g.replay()
            assert np.array_equal(b.accelerations(2), ref_a)
            with torch.cuda.stream(stream):
                for _ in range(3):
                    g.replay()
            for p, r in zip(b.get_state(2)[:3], ref[:3]):
                assert np.array_equal(p, r)
        b.sync()
