"""How many dense rows are copied beside a one-launch sort of more than 16384 pairs: more of them where shards begin
inside the shares of three or more wavefronts (of any, where the copies read nothing), which makes the sort longer.  Small integers:
every bit is fixed, whatever was copied."""
import pytest
import torch

from paper_1905_04035_amd import binding as ts
from paper_1905_04035_amd import workloads as wl

from parity import check, run_gpu, run_oracle
from test_epilogue_gpu import check_scaled

pytestmark = pytest.mark.gpu


def _rows_copied(V, d, lengths, dt=wl.ROW_FP32, dense=True):
    w = wl.make_custom(V=V, d=d, n_list=lengths, zipf_s=1.1, seed=V + d + len(lengths), row_dtype=dt, integer_values=True)
    g = run_gpu(w, mode="multi", dense=dense)
    check(g, run_oracle(w, dense=dense), w, exact_bits=True)
    assert g["info"]["sort_slices"] == 1
    return g["info"]["sort_copy_rows_end"]


@pytest.mark.parametrize("dt", [wl.ROW_FP32, wl.ROW_BF16])
def test_a_shard_that_begins_inside_a_share(dt):
    # 40000 pairs: shares of 2560; 48 MiB and 1.25 or 2.5 MiB per whole 1024 pairs beyond 16384, in work-groups of 256 KiB
    budget = lambda quarters: ((48 << 20) + 23 * (quarters << 18)) // (256 << 10) * 32
    for lengths in ([40000], [25600, 14400], [2560, 0, 37440], [40000, 0], [20000, 20000], [25601, 14399], [13333, 13333, 13334], [39999, 1],
                    [1, 0, 39999], [1, 1, 1, 1, 39996], [10000, 10000, 5600, 14400]):
        assert _rows_copied(32768, 1024, lengths, dt) == budget(5)
    for lengths in ([10000] * 4, [1, 2560, 2560, 34879], [13333, 13333, 1, 13332, 1], [5000] * 8):
        assert _rows_copied(32768, 1024, lengths, dt) == budget(10)


def test_a_shard_that_begins_inside_a_share_without_a_dense_operand():
    # as above in work-groups of 128 KiB
    budget = lambda quarters: ((48 << 20) + 23 * (quarters << 18)) // (128 << 10) * 32
    for lengths in ([40000], [25600, 14400], [40000, 0]):
        assert _rows_copied(32768, 1024, lengths, dense=False) == budget(5)
    for lengths in ([20000, 20000], [39999, 1], [13333, 13333, 13334], [5000] * 8):
        assert _rows_copied(32768, 1024, lengths, dense=False) == budget(10)


@pytest.mark.parametrize("V,d", [(60000, 64), (60000, 260), (45000, 128)])
@pytest.mark.parametrize("n", [1024, 5000, 16384])
def test_one_work_group_per_compute_unit_in_small_calls(V, d, n):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    G = -(-V // 512)
    for lengths in ([n], [n // 2 + 1, n - n // 2 - 1], [n // 9] * 8 + [n - n // 9 * 8]):          # begin inside shares
        wgs = (32 + n // 1024) * 4
        if 4 * (G + wgs) >= 3 * cus:
            wgs = cus - G
        assert _rows_copied(V, d, lengths) == min(V, wgs * 32768 // d)


@pytest.mark.parametrize("V,d,part", [(32768, 256, 512), (32768, 1024, 512), (9000, 1024, 128)])
@pytest.mark.parametrize("n", [16385, 18500, 22528, 22529, 27000])
def test_one_work_group_per_compute_unit_instead_of_a_few_more(V, d, part, n):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    G = -(-V // part)
    wgs = ((48 << 20) + (n - 16384) // 1024 * (5 << 18)) // (256 << 10)
    if G + wgs > cus and n <= 22528:
        wgs = cus - G
    for lengths in ([n], [n // 2 + 1, n - n // 2 - 1]):
        assert _rows_copied(V, d, lengths) == min(V, wgs * 32 * 1024 // d)
    # shards that begin inside three shares: the copies that the longer sort has room for
    wgs = ((48 << 20) + (n - 16384) // 1024 * (10 << 18)) // (256 << 10)
    assert _rows_copied(V, d, [n // 4 + 1] * 3 + [n - 3 * (n // 4 + 1)]) == min(V, wgs * 32 * 1024 // d)


@pytest.mark.parametrize("V,d,n", [(41900, 256, 65536), (32768, 512, 65536), (60000, 64, 58000), (60000, 64, 66000), (5000, 512, 60000)])
def test_copies_beside_a_sliced_sort(V, d, n):
    # 32 MiB beside each of the two launches up to four slices, 16 MiB up to six, but no more work-groups than
    # there are compute units that don't sort, unless the sort takes them all
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    S = -(-n // 16384)
    part = 2048 if -(-V // 2048) * S >= 256 else 1024
    idle = cus - -(-V // part) * S
    wgs = 128 if S <= 4 else 64
    wgs = min(wgs, idle) if idle > 0 else wgs
    w = wl.make_custom(V=V, d=d, n_list=[n], zipf_s=1.1, seed=V + d, integer_values=True)
    g = run_gpu(w, mode="multi")
    check(g, run_oracle(w), w, exact_bits=True)
    assert g["info"]["sort_slices"] == S
    assert g["info"]["sort_copy_rows_end"] == min(V, 2 * (wgs * 32768 // d))
    # an fp32 result without a dense operand: the whole budget, in half the bytes per row
    g = run_gpu(w, mode="multi", dense=False)
    check(g, run_oracle(w, dense=False), w, exact_bits=True)
    assert g["info"]["sort_copy_rows_end"] == min(V, 2 * ((256 if S <= 4 else 128) * 32768 // d))


@pytest.mark.parametrize("dense,out,elem_bytes", [(True, ts.TS_OUT_FP32, 8), (True, ts.TS_OUT_BF16, 6), (False, ts.TS_OUT_FP32, 4),
                                                  (False, ts.TS_OUT_BF16, 4)])
@pytest.mark.parametrize("n", [3000, 22528, 22529])
def test_the_budget_counts_bytes_that_move(monkeypatch, n, dense, out, elem_bytes):
    # a bf16 result without a dense operand counts as an fp32 one, except beside a long sort
    V, d = 40000, 1024
    seen, read_views = {}, ts.ts_read_views
    monkeypatch.setattr(ts, "ts_read_views", lambda *a: (seen.update(ts.ts_last_launch_info()), read_views(*a))[1])
    w = wl.make_custom(V=V, d=d, n_list=[n], zipf_s=1.1, seed=n, integer_values=True)
    check_scaled(w, 0.5, out, exact_bits=True, dense=dense)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    G = -(-V // 512)
    if n > 22528 and not dense and out == ts.TS_OUT_BF16:
        elem_bytes = 2
    budget = (32 << 20) + (n // 1024 << 20) if n <= 16384 else (48 << 20) + (n - 16384) // 1024 * (5 << 18)
    wgs = budget // (elem_bytes * 32768)
    if 4 * (G + wgs) >= 3 * cus and (G + wgs < cus or (dense and n <= 22528)):
        wgs = cus - G
    assert seen["sort_copy_rows_end"] == min(V, wgs * 32)
