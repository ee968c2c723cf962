"""The sort where its tables, lists and rounds can go wrong: sub-slices that end at and beside whole tiles and
rounds; ids that share a table word and take all pairs, in blocks and in turn; lists of owned pairs that
overflow; shards that begin anywhere inside a wavefront's share; the longest slice whose counts fit 16 bits and the
first that takes 32.  Small integers: every bit is fixed, and the sorted order is compared pair by pair."""
import numpy as np
import pytest

from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _workload(V, lengths, ids, seed):
    w = wl.make_custom(V=V, d=4, n_list=lengths, zipf_s=1.1, seed=seed, integer_values=True)
    rng = np.random.default_rng(seed)
    at = 0
    for a in w.ids:
        t = at + np.arange(len(a))
        if ids == "two in turn":                # ids of one table word
            a[:] = V // 4 * 2 + t % 2
        elif ids == "two blocks":
            a[:] = V // 4 * 2 + (t > sum(lengths) // 3)
        elif ids == "hot":                      # more of them than a list of owned pairs holds
            a[rng.random(len(a)) < 0.97] = V // 3
        elif ids == "some outside":
            a[rng.random(len(a)) < 0.2] = rng.choice([-1, -2 ** 31, V, 2 ** 31 - 1])
        at += len(a)
    return w


def _check(w, **kw):
    g = run_gpu(w, mode="multi", **kw)
    check(g, run_oracle(w), w, exact_bits=True)
    return g


@pytest.mark.parametrize("ids", ["zipf", "two in turn", "two blocks", "hot", "some outside"])
@pytest.mark.parametrize("n", [1, 63, 1025, 16383, 16384, 16385, 32768, 32769, 49153, 57344, 57345, 65536 + 1025])
def test_rounds(n, ids):
    for V in (700, 33000):
        _check(_workload(V, [n], ids, seed=n + V))


@pytest.mark.parametrize("ids", ["zipf", "hot"])
@pytest.mark.parametrize("n,k", [(999, 64), (16384, 3), (20001, 64), (57344, 5), (70001, 64)])
def test_shards_that_begin_anywhere(n, k, ids):
    rng = np.random.default_rng(n + k)
    cuts = np.sort(rng.integers(0, n + 1, k - 1))
    cuts[k // 2:k // 2 + 1] = cuts[k // 2 - 1] if k > 2 else cuts[0]          # an empty one among them
    lengths = np.diff(np.concatenate([[0], np.sort(cuts), [n]])).tolist()
    _check(_workload(5000, lengths, ids, seed=n + k))


@pytest.mark.parametrize("part", [64, 512, 2048])
def test_parts(part):
    ts.ts_set_sort_part(part)
    try:
        for n in (5000, 40000, 70000):
            for ids in ("zipf", "hot"):
                _check(_workload(20000, [n], ids, seed=part + n))
    finally:
        ts.ts_set_sort_part(0)


@pytest.mark.parametrize("n", [64 * 64512, 64 * 64512 + 1])
@pytest.mark.parametrize("ids", ["two in turn", "hot"])
def test_the_longest_slice_of_16_bits(n, ids):
    g = _check(_workload(3000, [n - 5, 5], ids, seed=3))
    assert g["info"]["sort_slices"] == 64           # of 64512 and (all but the last) of 65536 pairs
