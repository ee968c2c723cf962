"""Calls that take one launch: the limits of that form (pairs, pairs times lanes of a row, elements of the output, pairs times
elements) from both sides, widths at which a row takes 1, 2, 4 .. 64 lanes and several blocks of columns, vocabularies that end inside,
at and behind a work-group's rows, ids that leave long rows inside a group of pieces, across groups and across the whole
call; the same shapes beyond the limits in the two-launch form.  Normal data: the bits have to be those of the two-launch form, the sums within the stated bound of the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle
from test_epilogue_gpu import run_scaled
from test_range_gpu import check_range

pytestmark = pytest.mark.gpu


def _lanes(d):
    lanes = 1
    while lanes < 64 and lanes * 4 < d:
        lanes *= 2
    return lanes


def _pairs(d):
    return min(4096, 32768 // _lanes(d))


def _small(V, d, n):
    return 1 <= n <= 2048 and n * _lanes(d) <= 32768 and V * d <= 5 << 19 and V * d * n <= (13 if d <= 128 else 8) << 27


def _workload(V, d, n, dt=wl.ROW_FP32, ids="zipf", k=1):
    lengths = [n // k] * k
    lengths[-1] += n - sum(lengths)
    w = wl.make_custom(V=V, d=d, n_list=lengths, zipf_s=1.1, seed=V + d + n + len(ids), row_dtype=dt)
    rng = np.random.default_rng(V + n)
    for a in w.ids:
        if ids == "one":
            a[rng.random(len(a)) < 0.95] = V // 2
        elif ids == "few":
            a[:] = rng.integers(0, min(V, 5), len(a))
        elif ids == "uniform":
            a[:] = rng.integers(0, V, len(a))
        elif ids == "low":
            a[:] = rng.integers(0, min(V, 32), len(a))
        elif ids == "outside":
            a[rng.random(len(a)) < 0.3] = rng.choice([-1, V, 2 ** 31 - 1, -2 ** 31])
    return w


def _both(run):
    """run() as it is and with the two-launch form asked for."""
    got = run()
    ts.ts_set_short_rows(0)
    try:
        return got, run()
    finally:
        ts.ts_set_short_rows(-1)


def _check(w, **kw):
    r = run_oracle(w, dense=kw.get("dense", True))
    g, f = _both(lambda: run_gpu(w, mode="multi", **kw))
    assert (g["info"]["short_rows"] == 3) == _small(w.V, w.d, w.n_total) and f["info"]["short_rows"] == 0
    assert g["info"]["piece_tokens"] == f["info"]["piece_tokens"]
    check(g, r, w)
    assert np.array_equal(g["out"].view(np.uint32), f["out"].view(np.uint32))


@pytest.mark.parametrize("d", [4, 8, 12, 16, 32, 36, 64, 68, 128, 132, 256, 260, 512, 1028])
def test_widths_and_vocabularies(d):
    rows = 16 * 64 // _lanes(d)         # of a work-group in one round
    for V in (1, rows - 1, rows, rows + 1, 5 * rows + 3):
        for n in (1, 65, _pairs(d)):
            _check(_workload(V, d, n))


@pytest.mark.parametrize("ids", ["one", "few", "uniform", "outside"])
@pytest.mark.parametrize("d,V", [(4, 3000), (64, 1000), (64, 40960), (100, 20000), (128, 9000), (512, 700), (1024, 2000)])
def test_long_rows(d, V, ids):
    _check(_workload(V, d, _pairs(d), ids=ids))


@pytest.mark.parametrize("d", [20, 64, 68, 120, 300, 520])
def test_row_types_and_options(d):
    V = 900
    for dt in (wl.ROW_FP32, wl.ROW_BF16):
        for ids in ("zipf", "one"):
            w = _workload(V, d, _pairs(d) - 3, dt, ids, k=7)
            _check(w)
            _check(w, in_place=True)
            _check(w, dense=False)
            for out, in_place in ((ts.TS_OUT_FP32, False), (ts.TS_OUT_FP32, True), (ts.TS_OUT_BF16, False)):
                g, f = _both(lambda: run_scaled(w, 0.3, out, in_place=in_place)[0])
                assert np.array_equal(g.view(np.uint8), f.view(np.uint8))


def test_a_range_and_the_built_in_workspace(monkeypatch):
    seen, read_views = {}, ts.ts_read_views
    monkeypatch.setattr(ts, "ts_read_views", lambda *a: (seen.update(ts.ts_last_launch_info()), read_views(*a))[1])
    w = _workload(3000, 64, 2000, k=3)
    r = oracle.densify(w.ids, w.rows, 64, 3000, w.dense_in, wl.ROW_FP32)
    for v0, v1 in ((0, 100), (700, 1701), (2999, 3000)):
        check_range(w, r, v0, v1)
        assert seen["short_rows"] == 3
    ids, rows = (torch.from_numpy(t).cuda() for t in w.concatenated())
    dn = torch.from_numpy(w.dense_in).cuda()
    outs = _both(lambda: (lambda o: (ts.ts_densify_static(ids, rows, 64, 3000, dn, o), o.cpu().numpy())[1])(torch.empty_like(dn)))
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))


# one more pair than lets a row have 16, 8 or 4 lanes, 32 ids to a work-group and one more or fewer
@pytest.mark.parametrize("ids", ["one", "low", "zipf"])
@pytest.mark.parametrize("V,d,n", [(31, 64, 2048), (32, 64, 2048), (33, 64, 2047), (65, 60, 1025), (2000, 64, 1024), (2000, 68, 513), (2000, 68, 512),
                                   (6144, 64, 2048), (13312, 64, 2048), (26000, 64, 1048), (13600, 128, 1000), (2048, 1024, 512),
                                   (97, 1024, 512), (1500, 1024, 511), (97, 1028, 257), (10240, 256, 300)])
def test_columns_of_a_work_group(V, d, n, ids):
    assert _small(V, d, n)
    _check(_workload(V, d, n, ids=ids))
    _check(_workload(V, d, n, wl.ROW_BF16, ids, k=3), dense=n % 2 == 0)


@pytest.mark.parametrize("V,d,n,small", [(13312, 64, 2048, True), (13313, 64, 2048, False), (40960, 64, 665, True), (40960, 64, 666, False),
                                         (40961, 64, 300, False), (2048, 1024, 512, True), (2049, 1024, 512, False), (8192, 132, 512, True),
                                         (3000, 64, 2049, False), (3000, 68, 1024, True),
                                         (3000, 68, 1025, False), (3000, 128, 1024, True), (3000, 132, 512, True), (3000, 132, 513, False),
                                         (3000, 4, 2048, True), (3000, 4, 2049, False)])
def test_limits(V, d, n, small):
    assert small == _small(V, d, n)
    w = _workload(V, d, n)
    g = run_gpu(w, mode="multi")
    check(g, run_oracle(w), w)
    assert (g["info"]["short_rows"] == 3) == small


def test_replays_of_a_captured_call():
    w = _workload(2000, 64, 1500, ids="one")
    ids, rows = (torch.from_numpy(t).cuda() for t in w.concatenated())
    dn = torch.from_numpy(w.dense_in).cuda()
    ws = ts.Workspace(1500, 64, 2000)
    want, got = torch.empty_like(dn), torch.empty_like(dn)
    ts.ts_densify(ids, rows, 64, 2000, dn, want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ts.ts_densify(ids, rows, 64, 2000, dn, got)
    for _ in range(3):
        got.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        ts.ts_densify(ids, rows, 64, 2000, dn, want)
    ws.close()
