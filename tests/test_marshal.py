"""The binding's native marshalling: what it refuses (AssertionError before anything reaches the library, TypeError for
what is no tensor), and that lists, tuples, gradients and streams arrive as they are."""
import os

import numpy as np
import pytest
import torch

from paper_1905_04035_amd import binding as ts

V, D, N = 50, 8, 20


def _calls(dev, change=None):
    """(name, call) of every entry point on valid tensors, one of them put in place by change."""
    ids = torch.randint(V, (N,), dtype=torch.int32).to(dev)
    a = dict(ids=ids, rows=torch.ones(N, D, device=dev), dense_in=torch.zeros(V, D, device=dev),
             out=torch.empty(V, D, device=dev), rows16=torch.ones(N, D, dtype=torch.bfloat16, device=dev))
    if change:
        a.update({k: v for k, v in change(dict(a)).items()})
    i, r, h, x, o = a["ids"], a["rows"], a["rows16"], a["dense_in"], a["out"]
    return [("densify", lambda s=None: ts.ts_densify(i, r, D, V, x, o, s)),
            ("static", lambda s=None: ts.ts_densify_static(i, r, D, V, x, o, s)),
            ("bf16", lambda s=None: ts.ts_densify_bf16(i, h, D, V, x, o, s)),
            ("multi", lambda s=None: ts.ts_densify_multi([i], (r,), ts.TS_ROW_FP32, D, V, x, o, s)),
            ("scaled", lambda s=None: ts.ts_densify_scaled((i,), [r], ts.TS_ROW_FP32, D, V, x, o, 1.0, s)),
            ("range", lambda s=None: ts.ts_densify_range([i], [r], ts.TS_ROW_FP32, D, V, 0, V, x, o, s)),
            ("accumulate", lambda s=None: ts.ts_accumulate([("slices", i, r), ["dense", x]], ts.TS_RULE_PROPOSED, D, V, o, stream=s))]


def test_tensors_that_are_not_on_the_gpu_are_refused():
    for name, call in _calls("cpu"):
        with pytest.raises(AssertionError):
            call()


def test_what_is_no_tensor_or_no_sequence():
    t = torch.zeros(4, 4)
    for args in (([1], [t]), (1, [t]), ([t], None)):
        with pytest.raises(TypeError):
            ts.ts_densify_multi(*args, ts.TS_ROW_FP32, 4, 4, None, t)
    with pytest.raises(AssertionError):
        ts.ts_densify_multi([], [t], ts.TS_ROW_FP32, 4, 4, None, t)
    with pytest.raises(TypeError):
        ts.ts_densify("ids", t, 4, 4, None, t)
    with pytest.raises(AssertionError):
        ts.ts_accumulate([()], ts.TS_RULE_TF, 4, 4, t)


def test_iterators_are_no_sequences():
    t, i = torch.zeros(4, 4), torch.zeros(4, dtype=torch.int32)
    for ids_k, rows_k in ((iter([i]), [t]), ([i], iter([t])), ((x for x in [i]), (x for x in [t]))):
        with pytest.raises(TypeError):
            ts.ts_densify_multi(ids_k, rows_k, ts.TS_ROW_FP32, 4, 4, None, t)
        with pytest.raises(TypeError):
            ts.ts_densify_scaled(ids_k, rows_k, ts.TS_ROW_FP32, 4, 4, None, t, 1.0)
        with pytest.raises(TypeError):
            ts.ts_densify_range(ids_k, rows_k, ts.TS_ROW_FP32, 4, 4, 0, 4, None, t)
    for grads in (iter([("dense", t)]), [iter(("dense", t))]):
        with pytest.raises(TypeError):
            ts.ts_accumulate(grads, ts.TS_RULE_TF, 4, 4, t)


def test_calls_that_launch_nothing_do_without_the_module(monkeypatch):
    t, i = torch.zeros(4, 4), torch.zeros(4, dtype=torch.int32)
    monkeypatch.setattr(ts, "MARSHAL_PATH", os.path.join(os.path.dirname(ts.MARSHAL_PATH), "not_built.so"))
    monkeypatch.setattr(ts, "_marshal", None)
    monkeypatch.setattr(ts, "_lib", None)
    assert ts.ts_workspace_bytes(100, 64, 1000) > 0
    assert ts.ts_buffer_bytes(1, 1, 4, 1) == (20, 16)
    assert ts.ts_fusion_place(1 << 20, 1, 4, 1) == (256, 272)
    assert ts.status_string(ts.TS_ERR_SHAPE)
    for call in (lambda: ts.ts_densify(i, t, 4, 4, None, t), lambda: ts.ts_densify_multi([i], [t], ts.TS_ROW_FP32, 4, 4, None, t),
                 lambda: ts.ts_accumulate([("dense", t)], ts.TS_RULE_TF, 4, 4, t)):
        with pytest.raises(FileNotFoundError, match="not_built.so"):
            call()


@pytest.mark.gpu
@pytest.mark.parametrize("what,names", [
    (lambda a: dict(ids=a["ids"].long()), "all"), (lambda a: dict(ids=a["ids"].cpu()), "all"),
    (lambda a: dict(ids=torch.stack([a["ids"]] * 2, 1)[:, 0]), "all"),
    (lambda a: dict(rows=a["rows"].cpu()), "fp32"), (lambda a: dict(rows=a["rows"].half()), "fp32"),
    (lambda a: dict(rows=a["rows"].t().contiguous().t()), "fp32"), (lambda a: dict(rows=a["rows"][1:]), "fp32"),
    (lambda a: dict(rows16=a["rows16"].float()), "bf16"),
    (lambda a: dict(dense_in=a["dense_in"].double()), "all"), (lambda a: dict(dense_in=a["dense_in"][:, ::2]), "all"),
    (lambda a: dict(dense_in=a["dense_in"][1:]), "all"), (lambda a: dict(out=a["out"][1:]), "all"),
    (lambda a: dict(out=a["out"].double()), "all")])
def test_wrong_tensors_are_refused(what, names):
    ws = ts.Workspace(N, D, V)
    for name, call in _calls("cuda:0", what):
        if {"all": True, "fp32": name != "bf16", "bf16": name == "bf16"}[names]:
            with pytest.raises(AssertionError):
                call()
    ws.close()


@pytest.mark.gpu
def test_every_entry_point_on_streams():
    ws = ts.Workspace(N, D, V)
    side = torch.cuda.Stream()
    for name, call in _calls("cuda:0"):
        for stream in (None, side, torch.cuda.default_stream()):
            call(stream)
            torch.cuda.synchronize()
        with torch.cuda.stream(side):
            call()
        torch.cuda.synchronize()
    i = torch.randint(V, (N,), dtype=torch.int32, device="cuda:0")
    r = torch.ones(N, D, device="cuda:0")
    out = torch.empty(V, D, device="cuda:0")
    ts.ts_densify_multi((i[:7], i[7:]), [r[:7], r[7:]], ts.TS_ROW_FP32, D, V, None, out)
    want = np.bincount(i.cpu().numpy(), minlength=V).astype(np.float32)
    assert np.array_equal(out.cpu().numpy(), np.repeat(want[:, None], D, 1))
    ws.close()


def _gathered(**change):
    """A gather of two slice gradients and a dense one into outputs of exactly its size, or with some tensors replaced."""
    i = torch.randint(V, (N,), dtype=torch.int32, device="cuda:0")
    a = dict(ids=i, rows=torch.randn(N, D, device="cuda:0"), dense=torch.randn(V, D, device="cuda:0"), out=None,
             ids_out=torch.empty(2 * N + V, dtype=torch.int32, device="cuda:0"),
             rows_out=torch.empty(2 * N + V, D, device="cuda:0"))
    a.update({k: f(a[k]) for k, f in change.items()})
    grads = [("slices", a["ids"], a["rows"]), ("dense", a["dense"]), ("slices", a["ids"], a["rows"])]
    return a, ts.ts_accumulate(grads, ts.TS_RULE_TF, D, V, a["out"], a["ids_out"], a["rows_out"])


@pytest.mark.gpu
@pytest.mark.parametrize("change", [
    dict(ids_out=lambda t: t.cpu()), dict(ids_out=lambda t: t.long()), dict(ids_out=lambda t: torch.stack([t, t], 1)[:, 0]),
    dict(rows_out=lambda t: t.cpu()), dict(rows_out=lambda t: t.double()), dict(rows_out=lambda t: t[1:]),
    dict(rows_out=lambda t: t.t().contiguous().t()), dict(rows=lambda t: t[1:]), dict(dense=lambda t: t[1:])])
def test_wrong_tensors_of_a_gather_are_refused(change):
    with pytest.raises(AssertionError):
        _gathered(**change)


@pytest.mark.gpu
def test_accumulate_takes_flat_and_longer_buffers_and_leaves_unused_outputs_alone():
    def longer(t):
        return torch.cat([t, t])

    for change in (dict(), dict(rows=longer, dense=longer, ids_out=longer, rows_out=longer), dict(dense=lambda t: t.flatten()),
                   dict(rows=lambda t: t.flatten(), rows_out=lambda t: t.flatten()), dict(out=lambda t: torch.empty(3))):
        a, (strategy, total) = _gathered(**change)
        assert strategy == ts.TS_ACC_GATHER and total == 2 * N + V
        rows, dense = a["rows"].reshape(-1, D)[:N], a["dense"].reshape(-1, D)[:V]
        assert torch.equal(a["rows_out"].reshape(-1, D)[:total], torch.cat([rows, dense, rows]))
        ids = torch.cat([a["ids"], torch.arange(V, dtype=torch.int32, device="cuda:0"), a["ids"]])
        assert torch.equal(a["ids_out"][:total], ids)
    x = torch.randn(V, D, device="cuda:0")
    out = torch.empty(V * D + 5, device="cuda:0")
    for ids_out in (None, torch.empty(0), torch.empty(0, dtype=torch.int64, device="cuda:0")):
        assert ts.ts_accumulate([("dense", x), ("dense", x)], ts.TS_RULE_TF, D, V, out, ids_out) == (ts.TS_ACC_REDUCE, None)
        assert torch.equal(out[:V * D], (x + x).flatten())
    for shape in ((0, V), (D, 0), (-D, -V), (D + 1, V)):
        with pytest.raises(ts.TsError) as e:
            ts.ts_accumulate([("dense", longer(x))], ts.TS_RULE_TF, *shape, out)
        assert e.value.status == ts.TS_ERR_SHAPE
