"""Ranges of the vocabulary in calls whose sort takes several slices: small slices, the usual ones where
the tables of the small ones have no room or would take too many work-groups, groups of pieces beyond the
owned pairs, and a range that owns every pair although it has few of the ids.  Small integers: every bit
is fixed."""
import numpy as np
import pytest

import oracle
from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from test_range_gpu import check_range

pytestmark = pytest.mark.gpu


def _workload(V, d, n, dt, v0=0, v1=0):
    w = wl.make_custom(V=V, d=d, n_list=[n // 2, n - n // 2 - 77, 77], zipf_s=1.2, seed=V + d, row_dtype=dt,
                       integer_values=True)
    for a in w.ids if v1 else ():           # every pair into the range
        a[:] = v0 + a % (v1 - v0)
    return w


@pytest.mark.parametrize("V,d,n,dt,v0,v1,slices", [
    (9000, 64, 57345, wl.ROW_FP32, 0, 1000, 8), (9000, 64, 65537, wl.ROW_BF16, 1000, 1001, 9),
    (40000, 64, 131072, wl.ROW_FP32, 8193, 12290, 16), (40000, 60, 131073, wl.ROW_BF16, 39000, 40000, 17),
    (40000, 4, 131072, wl.ROW_FP32, 8193, 12290, 8),       # no room for the tables
    (60000, 64, 131072, wl.ROW_FP32, 0, 16385, 8),         # seventeen parts: more work-groups than compute units
    (9000, 64, 57344, wl.ROW_FP32, 0, 1000, 1)])
def test_slices(monkeypatch, V, d, n, dt, v0, v1, slices):
    seen, read_views = {}, ts.ts_read_views
    monkeypatch.setattr(ts, "ts_read_views", lambda *a: (seen.update(ts.ts_last_launch_info()), read_views(*a))[1])
    w = _workload(V, d, n, dt)
    check_range(w, oracle.densify(w.ids, w.rows, d, V, w.dense_in, dt), v0, v1, exact_bits=True)
    assert seen["sort_slices"] == slices


@pytest.mark.parametrize("dt", [wl.ROW_FP32, wl.ROW_BF16])
@pytest.mark.parametrize("n", [3000, 60000, 100000])
def test_a_small_range_with_every_pair(n, dt):
    w = _workload(20000, 64, n, dt, 5000, 5100)
    r = oracle.densify(w.ids, w.rows, 64, 20000, w.dense_in, dt)
    assert int(np.sum(r.count[5000:5100])) == n
    check_range(w, r, 5000, 5100, exact_bits=True)
