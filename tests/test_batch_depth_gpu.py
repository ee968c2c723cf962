"""How many value rows a wavefront of the pieces has in flight: the choice on both sides of each of its
limits, and the results there.  Small integers: every bit is fixed."""
import pytest

import oracle
from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle
from test_epilogue_gpu import check_scaled
from test_range_gpu import check_range

pytestmark = pytest.mark.gpu


def _depth(V, d, n, dt, **kw):
    w = wl.make_custom(V=V, d=d, n_list=[n - n // 3, n // 3], zipf_s=1.1, seed=V + d + n, row_dtype=dt, integer_values=True)
    g = run_gpu(w, mode="multi", **kw)
    check(g, run_oracle(w), w, exact_bits=True)
    assert g["info"]["short_rows"] == 0
    return g["info"]["deep_batches"]


# pairs per row up to which the batches are deep: fp32 rows in pieces of 16 and of 32, bf16 rows
@pytest.mark.parametrize("d,dt,n,limit", [(512, wl.ROW_FP32, 20000, 4), (256, wl.ROW_FP32, 96256, 4), (256, wl.ROW_FP32, 96257, 16),
                                          (256, wl.ROW_BF16, 40000, 8), (512, wl.ROW_BF16, 60000, 8)])
def test_many_pairs_per_row(d, dt, n, limit):
    V = -(-n // limit)
    assert _depth(V, d, n, dt) == 1
    assert _depth(V - 1, d, n, dt) == 0


@pytest.mark.parametrize("d,n", [(1024, 8192), (2048, 4096)])
def test_in_place_and_small_gathers(d, n):
    for pairs, deep in ((n, 1), (n + 1, 0)):
        assert _depth(700, d, pairs, wl.ROW_FP32) == deep             # many pairs per row
        assert _depth(4000, d, pairs, wl.ROW_FP32, in_place=True) == deep
        assert _depth(4000, d, pairs, wl.ROW_FP32) == 1


@pytest.mark.parametrize("V,d,dt,dense,deep", [
    (3000, 520, wl.ROW_FP32, True, 0), (3000, 520, wl.ROW_FP32, False, 0), (3000, 520, wl.ROW_BF16, True, 1), (65536, 384, wl.ROW_BF16, True, 1),
    (65537, 384, wl.ROW_BF16, True, 0), (65537, 512, wl.ROW_BF16, False, 1), (65537, 520, wl.ROW_BF16, False, 0)])
def test_a_bf16_result(monkeypatch, V, d, dt, dense, deep):
    seen, read_views = {}, ts.ts_read_views
    monkeypatch.setattr(ts, "ts_read_views", lambda *a: (seen.update(ts.ts_last_launch_info()), read_views(*a))[1])
    w = wl.make_custom(V=V, d=d, n_list=[5000, 4900], zipf_s=1.1, seed=V + d, row_dtype=dt, integer_values=True)
    check_scaled(w, 0.5, ts.TS_OUT_BF16, exact_bits=True, dense=dense)
    assert (seen["piece_tokens"], seen["short_rows"], seen["deep_batches"]) == (16, 0, deep)


# a range is taken to own its share of the pairs (rounded down), whatever it really owns
@pytest.mark.parametrize("V,d,dt,n,v0,v1,deep", [
    (9000, 512, wl.ROW_FP32, 36000, 1000, 6000, 1), (9000, 512, wl.ROW_FP32, 36002, 1000, 6000, 0),
    (9000, 512, wl.ROW_FP32, 36001, 0, 9000, 0), (32768, 256, wl.ROW_FP32, 131072, 8193, 12290, 1),
    (32767, 256, wl.ROW_FP32, 131073, 8193, 12290, 1), (6500, 1024, wl.ROW_BF16, 52000, 0, 1700, 1),
    (6500, 1024, wl.ROW_BF16, 52008, 0, 1700, 0)])
def test_ranges(monkeypatch, V, d, dt, n, v0, v1, deep):
    seen, read_views = {}, ts.ts_read_views
    monkeypatch.setattr(ts, "ts_read_views", lambda *a: (seen.update(ts.ts_last_launch_info()), read_views(*a))[1])
    for into_range in (False, True):
        w = wl.make_custom(V=V, d=d, n_list=[n // 2, n - n // 2], zipf_s=1.1, seed=V + d + n, row_dtype=dt, integer_values=True)
        if into_range:
            for a in w.ids:
                a[:] = v0 + a % (v1 - v0)
        check_range(w, oracle.densify(w.ids, w.rows, d, V, w.dense_in, dt), v0, v1, exact_bits=True)
        assert (seen["short_rows"], seen["deep_batches"]) == (0, deep)


@pytest.mark.parametrize("d,dt,limit", [(64, wl.ROW_FP32, 49152), (128, wl.ROW_FP32, 49152), (132, wl.ROW_FP32, 65536),
                                        (64, wl.ROW_BF16, 65536), (248, wl.ROW_BF16, 65536)])
def test_narrow_rows_in_large_numbers(d, dt, limit):
    V = limit // 2          # two pairs per row
    assert _depth(V, d, limit, dt) == 1
    assert _depth(V, d, limit + 1, dt) == 0
