"""Tuning a batch with split members: what a cached result holds for, and that
every candidate's time counts all of the members' pair sums."""
import json

import numpy as np
import pytest

from paper_2205_06557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


def _batch(B, n, kind=None):
    b = B.Batch([W.single_grain_small().with_(n_ions=n + 10 * k, system_id=k) for k in range(2)])
    if kind is not None:
        b.set_pair_kernel(kind)
    return b


def _lines(path):
    with open(path) as f:
        return [json.loads(x) for x in f]


def test_cache_tells_split_batches_apart(B, tmp_path):
    cache = str(tmp_path / "tune.jsonl")
    # the same sizes to a power of two; from 40,960 ions on members are split
    wanted = [(60000, None, 1), (60000, B.PAIR_SYMMETRIC, 2), (33000, None, 2), (60000, None, 2),
              (60000, B.PAIR_SYMMETRIC, 2)]
    ms = []
    for n, kind, lines in wanted:
        with _batch(B, n, kind) as b:
            ms.append(b.autotune(cache))
            assert len(_lines(cache)) == lines, (n, kind)
    keys = [x["key"] for x in _lines(cache)]
    assert len(set(keys)) == 2
    assert ms[3] == pytest.approx(ms[0], rel=1e-4) and ms[4] == pytest.approx(ms[1], rel=1e-4)


def test_tuning_after_a_one_sided_result(B, tmp_path):
    cache = str(tmp_path / "tune.jsonl")
    with _batch(B, 60000) as b:
        ref = b.autotune(cache)
    with open(cache) as f:
        line = f.read().replace('"symmetric": 1', '"symmetric": 0')
    with open(cache, "w") as f:
        f.write(line)
    with _batch(B, 60000) as b, _batch(B, 60000) as plain:
        b.autotune(cache)
        assert b.pair_kernel() == B.PAIR_ONE_SIDED
        ms = b.autotune(None)
        # timed without the split members' sums, candidates would take next to nothing
        assert ms > 0.5 * ref
        b.set_pair_kernel(B.PAIR_AUTO)
        for x in (b, plain):
            x.step(2)
            x.sync()
        for k in range(2):
            assert np.array_equal(b.accelerations(k), plain.accelerations(k))
