"""The length of the pieces fixes the order in which a row's pairs are added.  The library may choose it by
the pairs, the width, the row type and the vocabulary only: a call gives the same bits in place and out of
place, with its short rows added up in the pieces and row by row, through every entry point, and -- for rows
of few enough pairs that no piece cuts them -- as a range of the vocabulary.  Normal data, in which another
order of additions shows, at shapes where pieces of 8 are chosen and beside their limits."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle, to_dev
from test_epilogue_gpu import run_scaled
from test_range_gpu import check_range

pytestmark = pytest.mark.gpu

# (V, d, row type, pairs, pieces)
SHAPES = [(4000, 256, wl.ROW_FP32, 2000, 8), (2000, 512, wl.ROW_BF16, 12000, 8), (1000, 64, wl.ROW_FP32, 2048, 8),
          (12288, 1024, wl.ROW_FP32, 3000, 8), (12289, 1024, wl.ROW_FP32, 3000, 16), (32768, 1024, wl.ROW_FP32, 3000, 16),
          (40960, 512, wl.ROW_BF16, 12000, 8), (40961, 512, wl.ROW_BF16, 12000, 16), (4096, 512, wl.ROW_BF16, 32769, 16),
          (4000, 256, wl.ROW_FP32, 18433, 16), (12000, 516, wl.ROW_BF16, 9000, 16)]


def _workload(V, d, dt, n):
    return wl.make_custom(V=V, d=d, n_list=[n - n // 3, n // 3], zipf_s=1.1, seed=V + d + n, row_dtype=dt)


@pytest.mark.parametrize("V,d,dt,n,piece", SHAPES)
def test_the_same_bits_however_the_work_is_spread(V, d, dt, n, piece):
    w = _workload(V, d, dt, n)
    r = run_oracle(w)
    assert int(r.count.max()) > 4 * 64          # rows over several groups of pieces among them
    g = run_gpu(w, mode="multi")
    assert g["info"]["piece_tokens"] == piece
    check(g, r, w)
    want = g["out"].view(np.uint32)
    for mode in (0, 1):
        ts.ts_set_short_rows(mode)
        try:
            f = run_gpu(w, mode="multi")
        finally:
            ts.ts_set_short_rows(-1)
        assert f["info"]["piece_tokens"] == piece
        assert np.array_equal(f["out"].view(np.uint32), want), "short rows in the pieces / row by row"
    assert np.array_equal(run_gpu(w, mode="multi", in_place=True)["out"].view(np.uint32), want), "in place"
    assert np.array_equal(run_gpu(w, mode="single")["out"].view(np.uint32), want), "one buffer"
    assert np.array_equal(run_scaled(w, 1.0, ts.TS_OUT_FP32)[0].view(np.uint32), want), "scaled by 1"
    halved = run_scaled(w, 0.5, ts.TS_OUT_FP32, in_place=True)[0]
    assert np.array_equal(halved.view(np.uint32), (want.view(np.float32) * np.float32(0.5)).view(np.uint32)), "halved"
    if dt == wl.ROW_FP32 and ts.ts_workspace_bytes(n, d, V) <= ts.TS_STATIC_SCRATCH_BYTES:
        ids, rows = w.concatenated()
        out = torch.empty(V, d, device="cuda:0")
        ts.ts_densify_static(to_dev(ids), to_dev(rows), d, V, to_dev(w.dense_in), out)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want), "built-in workspace"


@pytest.mark.parametrize("V,d,dt,n,piece", SHAPES + [(20000, 1024, wl.ROW_FP32, 20000, 16), (9000, 64, wl.ROW_FP32, 100000, 32)])
def test_short_rows_of_a_range_have_the_bits_of_the_whole_call(V, d, dt, n, piece):
    w = _workload(V, d, dt, n)
    r = oracle.densify(w.ids, w.rows, d, V, w.dense_in, dt)
    g = run_gpu(w, mode="multi")
    assert g["info"]["piece_tokens"] == piece
    whole = g["out"].view(np.uint32)
    for v0, v1 in ((0, V // 8), (V // 3, V // 3 + 100), (V // 2, V)):
        part = check_range(w, r, v0, v1)["out"].view(np.uint32)
        short = r.count[v0:v1] <= piece
        assert np.array_equal(part[short], whole[v0:v1][short])
