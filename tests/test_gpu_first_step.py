"""od_step only queues work: the first step of a system whose pair sum needs no
further memory returns while the stream is still busy with what came before."""
import numpy as np
import pytest

from paper_2205_06557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ions,precision", [(2000, "FP64"), (20000, "FP64"), (100003, "FP64"), (2000, "FP32"),
                                              (30000, "FP32")])
def test_first_step_does_not_wait(n_ions, precision):
    import torch
    from paper_2205_06557_amd import binding as B
    w = W.single_grain_small().with_(n_ions=n_ions)
    prec = getattr(B, "PREC_" + precision)
    stream = torch.cuda.Stream()
    a = torch.ones((8192, 8192), device="cuda")
    torch.cuda.synchronize()
    with B.System(w, precision=prec, stream=stream.cuda_stream) as s, B.System(w, precision=prec) as ref:
        with torch.cuda.stream(stream):
            for _ in range(40):                 # about 0.3 s of work ahead of the step
                b = a @ a
            done = torch.cuda.Event()
            done.record(stream)
        s.step(1)
        assert not done.query()
        s.step(2)
        s.sync()
        assert done.query() and float(b[0, 0]) == 8192.0
        ref.step(3)
        for p, q in zip(s.get_state()[:3], ref.get_state()[:3]):
            assert np.array_equal(p, q)


@pytest.mark.parametrize("n_ions", [500, 12345, 60000])
def test_fp64_without_room_for_its_totals(n_ions):
    """Refused memory: totals and work items together, then either alone."""
    from paper_2205_06557_amd import binding as B
    w = W.single_grain_small().with_(n_ions=n_ions)
    acc = []
    for refuse in ((), (0,), (0, 2), (0, 3)):
        alloc = B.TorchAllocator()
        give, calls = alloc._a, []

        def some(ctx, nbytes):
            calls.append(int(nbytes))
            return None if len(calls) - 1 in refuse else give(ctx, nbytes)

        # calls: 0 everything, 1 the state alone, 2 the totals, 3 the work items
        hook = B.ALLOC_FN(some)
        alloc._a, alloc.struct = hook, B.Allocator(hook, alloc._f, None)
        real, B.TorchAllocator = B.TorchAllocator, lambda: alloc
        try:
            s = B.System(w, precision=B.PREC_FP64, torch_memory=True)
        finally:
            B.TorchAllocator = real
        with s:
            assert len(calls) == {(): 1, (0,): 4, (0, 2): 3, (0, 3): 4}[refuse]
            s.step(2)
            s.sync()
            acc.append(s.accelerations())
    assert np.array_equal(acc[0], acc[1])       # in the state's memory or apart
    assert np.array_equal(acc[2], acc[3])       # one-sided
    d = np.linalg.norm(acc[2] - acc[0], axis=0) / np.linalg.norm(acc[0], axis=0)
    assert np.median(d) < 1e-14 and d.max() < 1e-9
