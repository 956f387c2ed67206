"""The tuner's cache: a choice is kept for its device, engine and batch, and one
measured on another engine is not returned."""
import json

import pytest

import qaoa_inputs as qi
from paper_2407_13012_amd import batch_tune as bt


@pytest.fixture
def timed(monkeypatch):
    import torch
    calls = []
    monkeypatch.setattr(bt, "device_key", lambda: "dev|cu4")
    monkeypatch.setattr(bt, "_time_run", lambda graphs, p, g0, b0, steps, **opt: calls.append(opt) or float(len(calls)))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: type("Props", (), {"multi_processor_count": 4, "gcnArchName": "dev"}))
    return calls


def test_choices_of_another_engine_are_measured_again(tmp_path, timed, monkeypatch):
    cache = str(tmp_path / "cache.json")
    graphs = [qi.erdos_renyi(n, 0.5, seed=[1, n]) for n in (10, 14)]
    old = {"group_by_n": {}, "waves_per_simd": 2, "workgroups": 7, "resident_max_n": 0}
    with open(cache, "w") as fh:
        json.dump({"dev|cu4": {bt.batch_key(graphs, 2): old}}, fh)
    first = bt.tune(graphs, 2, cache=cache)
    assert timed and first["workgroups"] != 7
    count = len(timed)
    assert bt.tune(graphs, 2, cache=cache) == first and len(timed) == count
    monkeypatch.setattr(bt, "ENGINE", bt.ENGINE + 1)
    bt.tune(graphs, 2, cache=cache)
    assert len(timed) == 2 * count
