"""Calls with few pairs: pieces of 8 or of 16 sorted positions, half or all of a batch's value rows in
flight -- one size below, at and above each limit of the choice, with rows that lie inside a piece, span
the pieces of a group and span several groups, and small-integer values so that every bit is fixed."""
import pytest

from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import TOL, check, error_bound, run_gpu, run_oracle
from test_epilogue_gpu import check_scaled

pytestmark = pytest.mark.gpu


def _workload(V, d, n, dt, hot=()):
    w = wl.make_custom(V=V, d=d, n_list=[n - n // 3, n // 3], zipf_s=1.2, seed=V + d + n, row_dtype=dt, integer_values=True)
    at = 0
    for i, m in enumerate(hot):             # id 7 i of the first shard: m pairs
        w.ids[0][at:at + m] = 7 * i
        at += m
    return w


@pytest.mark.parametrize("V,d,dt,n,piece", [
    (3000, 1024, wl.ROW_FP32, 4096, 8), (3000, 1024, wl.ROW_FP32, 4097, 16),
    (5120, 1024, wl.ROW_FP32, 4608, 8), (5119, 1024, wl.ROW_FP32, 4608, 16), (5120, 1024, wl.ROW_FP32, 4609, 16), (12288, 1024, wl.ROW_FP32, 500, 8),
    (12289, 1024, wl.ROW_FP32, 500, 16), (3000, 64, wl.ROW_FP32, 16384, 8), (3000, 64, wl.ROW_FP32, 16385, 16),
    (1000, 260, wl.ROW_FP32, 8192, 8), (1000, 260, wl.ROW_FP32, 8193, 16), (20172, 260, wl.ROW_FP32, 9216, 8),
    (20172, 260, wl.ROW_FP32, 9217, 16), (1000, 516, wl.ROW_FP32, 6145, 16),
    (2000, 512, wl.ROW_BF16, 32768, 8), (2000, 512, wl.ROW_BF16, 32769, 16), (2000, 520, wl.ROW_BF16, 900, 16),
    (2000, 516, wl.ROW_BF16, 900, 16), (5000, 128, wl.ROW_FP32, 65536, 16), (5000, 128, wl.ROW_FP32, 65537, 16),
    (5000, 128, wl.ROW_BF16, 65537, 16), (5, 4, wl.ROW_FP32, 1, 8)])
def test_around_the_limits(V, d, dt, n, piece):
    w = _workload(V, d, n, dt)
    g = run_gpu(w, mode="multi")
    assert g["info"]["piece_tokens"] == piece
    check(g, run_oracle(w), w, exact_bits=True)


@pytest.mark.parametrize("V,d,n,dt", [(1000, 64, 2048, wl.ROW_FP32), (4000, 256, 16000, wl.ROW_FP32),
                                      (2000, 512, 30000, wl.ROW_BF16), (300, 264, 30000, wl.ROW_BF16)])
@pytest.mark.parametrize("s", [1.1, 1.8])
def test_measured_error_stays_under_the_a_priori_bound(V, d, n, dt, s):
    w = wl.make_custom(V=V, d=d, n_list=[n - n // 3, n // 3], zipf_s=s, seed=V + n, row_dtype=dt)
    g, r = run_gpu(w, mode="multi"), run_oracle(w)
    assert g["info"]["piece_tokens"] == 8
    bound = error_bound(int(r.count.max()), 8)
    worst = check(g, r, w)
    assert worst <= bound < TOL, (worst, bound)


@pytest.mark.parametrize("n", [8191, 8192, 8193])
def test_in_place_around_the_limit(n):
    w = _workload(3000, 1024, n, wl.ROW_FP32)
    check_scaled(w, 1.0, ts.TS_OUT_FP32, exact_bits=True, in_place=True)


@pytest.mark.parametrize("d,dt", [(64, wl.ROW_FP32), (260, wl.ROW_FP32), (64, wl.ROW_BF16), (264, wl.ROW_BF16)])
@pytest.mark.parametrize("hot", [(7, 8, 9, 15, 16, 17), (55, 56, 57, 63, 64, 65), (127, 128, 129, 1100)])
@pytest.mark.parametrize("out", [ts.TS_OUT_FP32, ts.TS_OUT_BF16])
def test_rows_across_pieces_and_groups(d, dt, hot, out):
    w = _workload(600, d, 2600, dt, hot)
    g = run_gpu(w, mode="multi")
    assert g["info"]["piece_tokens"] == 8
    check(g, run_oracle(w), w, exact_bits=True)
    check_scaled(w, 0.5, out, exact_bits=True)
