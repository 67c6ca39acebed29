"""Cached tunings of the autotuners: those chosen for other kernels are not
taken, on either path, and an unreadable cache is none."""
import json
import types

import paper_2210_00389_amd.batch as batch
import paper_2210_00389_amd.tune as tune


def _graph():
    return types.SimpleNamespace(n=1 << 18, nnz=1 << 22, cols=types.SimpleNamespace(device="cpu"))


def _batch():
    return types.SimpleNamespace(num_graphs=4, total_vertices=1000, total_nnz=8000,
                                 cols=types.SimpleNamespace(device="cpu"))


def test_only_tunings_of_the_present_kernels(tmp_path, monkeypatch):
    path = str(tmp_path / "autotune.json")
    monkeypatch.setattr(tune, "_cache_path", lambda: path)
    monkeypatch.setattr(batch, "_cache_path", lambda: path)
    gkey, bkey = tune.graph_key(_graph(), "cover"), batch.shape_key(_batch())

    class Searched(Exception):
        pass

    def search(*a, **k):
        raise Searched

    monkeypatch.setattr(tune, "Workspace", search)
    monkeypatch.setattr(batch, "Workspace", search)
    monkeypatch.setattr(batch.torch.cuda, "current_stream", lambda *a: None)

    def got(fn, arg):
        try:
            return fn(arg)
        except Searched:
            return "searched"

    for kernels, taken in ((None, False), ("another", False), (batch.kernels_id(), True)):
        e = dict(tuning=dict(item_log2=16), ms=1.0)
        if kernels:
            e["kernels"] = kernels
        json.dump({gkey: e, bkey: dict(e, tuning=dict(batch_piece=4096))}, open(path, "w"))
        assert got(tune.autotune_count, _graph()) == (dict(item_log2=16) if taken else "searched")
        assert got(batch.autotune, _batch()) == (dict(batch_piece=4096) if taken else "searched")
    for text in ("", "[1]", "{"):
        open(path, "w").write(text)
        assert got(tune.autotune_count, _graph()) == "searched"


def test_stored_tunings_are_found(tmp_path):
    path = str(tmp_path / "a" / "autotune.json")
    cache = batch.load_tunings(path)
    assert cache == {}
    batch.store_tuning(path, cache, "k", tuning=dict(batch_block=64), ms=2.0)
    assert batch.load_tunings(path)["k"]["tuning"] == dict(batch_block=64)
