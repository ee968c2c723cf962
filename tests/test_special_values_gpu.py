"""Signed zeros, NaN payloads, infinities, subnormals and the largest finite numbers, in every form of the kernels: rows without
pairs by each way of copying them, and infinities and NaN in the value rows and in dense_in of short and long rows (rows that end inside
a piece, a group of pieces, and over two levels of the tree).  Infinities are the same however a sum is ordered."""
import numpy as np
import pytest

from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import TOL, check, run_gpu, run_oracle
from test_epilogue_gpu import check_scaled
from test_random_shapes_gpu import _draw

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["beside the sort", "behind it", "row by row"])
def copies(request):
    """How rows without pairs are copied: copy_flat, copy_narrow or (wide rows) copy_chunk, short_row; all in two launches."""
    ts.ts_set_overlap_bytes(400 << 20 if request.param == "beside the sort" else 0)
    ts.ts_set_short_rows(1 if request.param == "row by row" else 0)
    yield request.param
    ts.ts_set_overlap_bytes(-1)
    ts.ts_set_short_rows(-1)


@pytest.mark.parametrize("V,d,n", [(100, 64, 30), (700, 4, 30), (300, 260, 40), (90, 516, 30), (60, 1028, 20), (40, 4100, 15)])
def test_rows_without_pairs(copies, V, d, n):
    w = wl.make_custom(V=V, d=d, n_list=[n], ids="distinct", seed=V + d)
    bits = w.dense_in.view(np.uint32)
    rng = np.random.default_rng(V)
    plain = bits.copy()
    bits[:, rng.permutation(d)[:4]] = [0x80000000, 0x7FC12345, 0xFF800000, 0x7F812345]
    g, r = run_gpu(w), run_oracle(w)
    assert g["info"]["short_rows"] == (1 if copies == "row by row" else 0)
    assert g["info"]["sort_copy_rows_end"] == (V if copies == "beside the sort" else 0)
    untouched = r.count == 0
    assert np.array_equal(g["out"][untouched].view(np.uint32), bits[untouched])
    assert np.array_equal(np.isnan(g["out"]), np.isnan(r.out))
    bits[:] = plain
    u = np.setdiff1d(np.arange(V), w.ids[0])
    bits[u[:, None], rng.permutation(d)[:4]] = [0x80000000, 0xFF800000, 0x00000001, 0x7F7FFFFF]
    check_scaled(w, 0.5, ts.TS_OUT_FP32)
    check_scaled(w, 0.5, ts.TS_OUT_FP32, in_place=True)
    check_scaled(w, 1.0, ts.TS_OUT_BF16)
    check_scaled(w, -1.5, ts.TS_OUT_BF16)


def _row_counts(V, d, counts, dt, seed):
    """Row 3 + 2 i receives counts[i] pairs, in shuffled order.  Every other one of them has infinities and NaN: in some of its
    columns, the first and the last among them, one pair's value, two pairs' of opposite signs, or dense_in's."""
    rng = np.random.default_rng(seed)
    ids = np.concatenate([np.full(c, 3 + 2 * i, np.int32) for i, c in enumerate(counts)])
    ids = ids[rng.permutation(len(ids))]
    rows = rng.normal(size=(len(ids), d)).astype(np.float32)
    dense = rng.normal(size=(V, d)).astype(np.float32)
    if dt == wl.ROW_BF16:
        rows = ((wl.fp32_to_bf16_bits(rows).astype(np.uint32)) << 16).view(np.float32)
    for i, c in enumerate(counts):
        if i % 2 == 0:
            t = np.flatnonzero(ids == 3 + 2 * i)[[0, -1, c // 2, (7 * i) % c]]
            rows[t[i // 2 % 4], 0] = np.inf
            rows[t[3], 1] = np.nan
            rows[t[1], 2] = -np.inf
            rows[t[0], d // 2] = np.inf
            rows[t[1], d // 2] = -np.inf if c > 1 else np.inf
            rows[t[2], d - 1] = -np.inf
            dense[3 + 2 * i, d - 2] = np.inf
    if dt == wl.ROW_BF16:
        rows = (rows.view(np.uint32) >> 16).astype(np.uint16)
    return wl.Workload(spec=wl.Spec("custom", -1, V, d, 1, 0, "zipf", row_dtype=dt), ids=[ids], rows=[rows], dense_in=dense)


FEW = [1, 2, 7, 8, 9, 15, 16, 17, 18, 31, 40, 64, 65, 70, 130, 131, 300, 300]
MANY = FEW + [900, 901, 1300, 4000, 2500]


@pytest.mark.parametrize("form", ["chosen", "in the pieces", "row by row"])
@pytest.mark.parametrize("dt", [wl.ROW_FP32, wl.ROW_BF16])
@pytest.mark.parametrize("V,d,counts", [(60, 64, FEW), (60, 20, FEW), (60, 260, FEW[:14]), (60, 1040, FEW[:15]), (500, 512, MANY), (3000, 1032, MANY),
                                        (60, 256, [30000, 20000, 9] * 2), (60, 256, [40000, 25000, 9] * 2)])
def test_infinities_and_nan_in_sums(V, d, counts, dt, form):
    w = _row_counts(V, d, counts, dt, V + d + len(counts))
    r = run_oracle(w)
    ts.ts_set_short_rows({"chosen": -1, "in the pieces": 0, "row by row": 1}[form])
    try:
        g = run_gpu(w)
    finally:
        ts.ts_set_short_rows(-1)
    assert (g["info"]["short_rows"] == 3) == (form == "chosen" and V == 60 and sum(counts) <= 512 * 1040 // d and sum(counts) <= 2048)
    assert np.array_equal(g["count"], r.count)
    assert np.array_equal(np.isnan(g["out"]), np.isnan(r.exact))
    inf = np.isinf(r.exact)
    assert inf.sum() >= 4 * ((len(counts) + 1) // 2) and np.array_equal(np.where(inf, g["out"], 0), np.where(inf, r.exact, 0))
    fin = np.isfinite(r.exact)
    assert (np.abs(g["out"][fin] - r.exact[fin]) <= TOL * r.abs_sum[fin]).all()


@pytest.mark.parametrize("rule", [0, 1])
def test_empty_and_ragged_shards_in_two_launches(rule):
    w = wl.make_custom(V=900, d=128, n_list=[0, 70, 0, 1, 64, 129, 0], seed=44)
    ts.ts_set_short_rows(rule)
    try:
        a, b = run_gpu(w, mode="multi"), run_gpu(w, mode="single")
    finally:
        ts.ts_set_short_rows(-1)
    assert a["info"]["short_rows"] == rule
    check(a, run_oracle(w), w)
    assert np.array_equal(a["out"].view(np.uint32), b["out"].view(np.uint32)) and np.array_equal(a["perm"], b["perm"])


@pytest.mark.parametrize("seed", [s for s in range(160) if sum(_draw(s)[0]["n_list"]) <= 4097])
def test_random_shapes_of_small_calls_in_two_launches(seed):
    kw, rng = _draw(seed)
    w = wl.make_custom(integer_values=True, **kw)
    ts.ts_set_short_rows(seed % 2)
    try:
        g = run_gpu(w, mode="multi", dense=seed % 3 > 0, in_place=seed % 3 == 2)
    finally:
        ts.ts_set_short_rows(-1)
    assert g["info"]["short_rows"] != 3
    check(g, run_oracle(w, dense=seed % 3 > 0), w, exact_bits=True)
