"""The autotuner's cache keys (host code) name the grouping of the launches that the times
are of: entries of other kernels are not taken."""

import json
from types import SimpleNamespace

import torch

from paper_1411_4283_amd import api


def _builder(monkeypatch):
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: SimpleNamespace(gcnArchName="gfx950:sramecc+:xnack-"))
    b = object.__new__(api.Builder)
    b.dim, b.device, b.built = 3, "cuda", 0
    b.opts = SimpleNamespace(order=4, path_radius=3, tuning=None)

    def build(out=None, stream=None):
        b.built += 1

    b.build = build
    counts = [0, 0, 0, 10, 20, 30, 0, 0]

    def last_bin_faces(c, n):
        c[:] = counts
        return 8

    monkeypatch.setattr(api, "load", lambda: SimpleNamespace(cutcell_last_bin_faces=last_bin_faces))
    return b


def test_entries_without_the_launch_version_are_not_taken(tmp_path, monkeypatch):
    b = _builder(monkeypatch)
    path = str(tmp_path / "t.json")
    entry = {"xcd_chunks": 8, "blocks_per_xcd": 128, "split": 2, "best_ms": 1.5}
    with open(path, "w") as fh:   # as kept when every bin had launches and kernel widths of its own
        json.dump({f"gfx950/D3/Q4/R3/bin{i}": entry for i in range(8)}, fh)
    assert b._tuning_from_cache(path, None, None) is None
    t = api.Tuning()
    for i in range(8):
        t.xcd_chunks[i], t.blocks_per_xcd[i] = 8, 0
    api._cache_store(path, b._cache_prefix(), t, [-1.0, -1.0, -1.0, 0.1, 0.2, 0.2, -1.0, -1.0])
    got = b._tuning_from_cache(path, None, None)
    assert got is not None and list(got.xcd_chunks) == [0, 0, 0, 8, 8, 8, 0, 0] and not any(got.blocks_per_xcd)
