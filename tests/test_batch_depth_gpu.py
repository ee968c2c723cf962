"""How many value rows a wavefront of the pieces has in flight: the choice on both sides of each of its
limits, and the results there.  Small integers: every bit is fixed."""
import pytest

import oracle
from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle
from test_range_gpu import run_range, check_range

pytestmark = pytest.mark.gpu


def _depth(V, d, n, dt, **kw):
    w = wl.make_custom(V=V, d=d, n_list=[n - n // 3, n // 3], zipf_s=1.1, seed=V + d + n, row_dtype=dt, integer_values=True)
    g = run_gpu(w, mode="multi", **kw)
    check(g, run_oracle(w), w, exact_bits=True)
    assert g["info"]["short_rows"] == 0
    return g["info"]["deep_batches"]


@pytest.mark.parametrize("d,dt,limit", [(64, wl.ROW_FP32, 49152), (128, wl.ROW_FP32, 49152), (132, wl.ROW_FP32, 65536),
                                        (64, wl.ROW_BF16, 65536), (248, wl.ROW_BF16, 65536)])
def test_narrow_rows_in_large_numbers(d, dt, limit):
    V = limit // 2          # two pairs per row
    assert _depth(V, d, limit, dt) == 1
    assert _depth(V, d, limit + 1, dt) == 0
