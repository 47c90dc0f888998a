"""A launch setting saved when the modes meant other launches (0 one per level,
1 cooperative) is not applied: the tuners measure again."""
import importlib
import json
import types

import pytest
import torch

tune = importlib.import_module("paper_2606_18900_amd.tune")       # the package has a function of that name


class _Measures(Exception):
    pass


class _Arc:
    info = types.SimpleNamespace(n=1000, n_blocks=1, n_levels=1, source_fnv=-2, max_record_len=100)
    n, n_reads, device = 1000, 3, torch.device("cpu")

    def __init__(self):
        self.set = []

    def set_tuning(self, **kw):
        self.set.append(kw)

    def scratch_bytes(self, n):
        return 256

    def _measure(self, *a, **kw):
        raise _Measures

    decode_all = read_lookup = _measure


@pytest.mark.parametrize("what,fn,saved", [
    ("decode", tune.tune, dict(sync_mode=1, wg_per_cu=2, ms=1.0)),
    ("requests", tune.tune_requests, dict(req_sync_mode=1, plan_blocks=1, us=1.0))])
def test_saved_before_the_modes_changed(tmp_path, monkeypatch, what, fn, saved):
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda d: "dev")
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d: None)
    old = "%s|dev|n=1000|blocks=1|levels=1|fnv=%016x" % (what, 2 ** 64 - 2)
    path = tmp_path / "cache.json"
    path.write_text(json.dumps({old: saved}))
    arc = _Arc()
    with pytest.raises(_Measures):
        fn(arc, cache_path=str(path))
    # what is saved under the present key is applied
    path.write_text(json.dumps({tune._key(arc, what): saved}))
    assert fn(arc, cache_path=str(path))["cached"]
    assert arc.set[-1] == {k: v for k, v in saved.items() if k not in ("ms", "us")}
