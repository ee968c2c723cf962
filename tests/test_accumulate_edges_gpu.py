"""ts_accumulate where its launches change form: runs of a gather one element below, at and above a
work-group, more runs than one launch's table holds, and sums whose last work-group is partly
filled, for every number of sources that has a form of its own.  Copies and small integers: exact."""
import numpy as np
import pytest
import torch

from oracle import accumulate as acc
from paper_1905_04035_amd import binding as ts

from parity import DEV
from test_accumulate_gpu import _dev, _run

pytestmark = pytest.mark.gpu


def _slices(rng, n, d, V):
    return ("slices", rng.integers(0, V, size=n).astype(np.int32), rng.integers(-4, 5, size=(n, d)).astype(np.float32))


def _dense(rng, d, V):
    return ("dense", rng.integers(-4, 5, size=(V, d)).astype(np.float32))


@pytest.mark.parametrize("d,V,lengths", [
    (4, 63, [1, 63, 64, 65]), (4, 64, [0, 64, 1]), (4, 65, [127, 128, 129]), (260, 1000, [1, 3, 1021]),
    (8, 5, list(range(40))),                     # 82 runs: two launches
])
def test_gather_runs(d, V, lengths):
    rng = np.random.default_rng(d + V)
    grads = [_slices(rng, n, d, V) for n in lengths] + [_dense(rng, d, V)]
    r = acc.accumulate(grads, acc.RULE_TF, d, V)
    st, n, _, ids, rows = _run(grads, ts.TS_RULE_TF, d, V, sum(lengths))
    assert st == ts.TS_ACC_GATHER and n == len(r.ids)
    assert np.array_equal(ids[:n], r.ids) and np.array_equal(rows[:n], r.rows)
    assert np.all(ids[n:] == -7) and np.all(np.isnan(rows[n:]))


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 16])
@pytest.mark.parametrize("d,V", [(4, 1), (4, 255), (4, 1023), (4, 1024), (4, 1025), (516, 301)])
def test_sums(m, d, V):
    rng = np.random.default_rng(m * 10000 + V)
    grads = [_dense(rng, d, V) for _ in range(m)]
    r = acc.accumulate(grads, acc.RULE_PROPOSED, d, V)
    _, n, dense, _, _ = _run(grads, ts.TS_RULE_PROPOSED, d, V, 0)
    assert n is None and np.array_equal(dense, r.dense)


@pytest.mark.parametrize("n", [5, 64, 30000])
def test_a_gather_reads_ids_that_lie_in_its_output_before_it_writes_over_them(n):
    """A gradient's ids in the place where a later gradient's ids go, or where a later one's rows go: read
    before anything later is written.  Ids in their own place stay what they are."""
    d, V = 8, 1000
    rng = np.random.default_rng(n)
    grads = [_slices(rng, n, d, V) for _ in range(3)] + [_dense(rng, d, V)]
    r = acc.accumulate(grads, acc.RULE_TF, d, V)
    for place in ("ids of the second", "ids of the dense one", "rows of the third", "its own", "its own, the second's too"):
        ids_out = torch.full((3 * n + V,), -7, dtype=torch.int32, device=DEV)
        rows_out = torch.full((3 * n + V, d), float("nan"), dtype=torch.float32, device=DEV)
        gd = _dev(grads)
        at = {"ids of the second": ids_out[n:2 * n], "ids of the dense one": ids_out[3 * n + V - min(n, V):][:n],
              "rows of the third": rows_out[2 * n:3 * n].view(torch.int32).reshape(-1)[:n]}.get(place, ids_out[:n])
        if at.numel() < n:
            at = ids_out[2 * n:3 * n]
        at.copy_(gd[0][1])
        gd[0] = ("slices", at, gd[0][2])
        if "second's too" in place:
            ids_out[n:2 * n] = gd[1][1]
            gd[1] = ("slices", ids_out[n:2 * n], gd[1][2])
        _, total = ts.ts_accumulate(gd, ts.TS_RULE_TF, d, V, None, ids_out, rows_out)
        torch.cuda.synchronize()
        assert total == 3 * n + V
        assert np.array_equal(ids_out.cpu().numpy(), r.ids), place
        assert np.array_equal(rows_out.cpu().numpy(), r.rows), place
