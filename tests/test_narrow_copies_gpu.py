"""Copies of rows without pairs where a wavefront takes several narrow rows (d <= 512: 1024 / d, at most
64 rows), and the copies beside the sort, 2048 elements per wavefront whatever the rows' width: the
last wavefront partly filled, exactly filled, one row over; widths that divide 1024 and widths that do
not.  Small integers: every bit is fixed."""
import pytest

from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle
from test_epilogue_gpu import check_scaled

pytestmark = pytest.mark.gpu


def _workload(V, d, n):
    return wl.make_custom(V=V, d=d, n_list=[n - n // 3, n // 3], zipf_s=1.2, seed=V + d, integer_values=True)


@pytest.mark.parametrize("d", [4, 16, 20, 64, 252, 256, 260, 340, 344, 508, 512, 516])
def test_rows_per_wavefront(d):
    R = max(1, min(64, 1024 // d))
    for V in (1, R, 7 * R - 1, 7 * R, 7 * R + 1):
        w = _workload(V, d, 5)
        r = run_oracle(w)
        for overlap in (0, -1):          # every untouched row by the second launch; most of them beside the sort
            ts.ts_set_overlap_bytes(overlap)
            try:
                check(run_gpu(w, mode="single"), r, w, exact_bits=True)
                for out_dtype in (ts.TS_OUT_FP32, ts.TS_OUT_BF16):
                    check_scaled(w, 0.25, out_dtype, exact_bits=True)
                    check_scaled(w, 0.25, out_dtype, exact_bits=True, dense=False)
                check_scaled(w, 0.25, ts.TS_OUT_FP32, exact_bits=True, in_place=True)
            finally:
                ts.ts_set_overlap_bytes(-1)


@pytest.mark.parametrize("V,d", [(511, 4), (512, 4), (513, 4), (8192, 4), (8193, 4), (1639, 20), (40000, 260), (3000, 4096)])
@pytest.mark.parametrize("mib", [1, 16, 400])
def test_copies_beside_the_sort(V, d, mib):
    w = _workload(V, d, 700)
    ts.ts_set_overlap_bytes(mib << 20)
    try:
        check(run_gpu(w, mode="single"), run_oracle(w), w, exact_bits=True)
    finally:
        ts.ts_set_overlap_bytes(-1)
