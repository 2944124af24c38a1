"""Picks of other kernels in the autotuner's cache are not replayed (no device: an
entry that is used is returned before any trial)."""
import json
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1002_1202_amd import autotune


class Trial(Exception):
    pass


def test_old_entries_are_not_replayed(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("GSC_AUTOTUNE_CACHE", str(path))
    pair = SimpleNamespace(block=4, n=4096)
    z, rhs = np.zeros(64, complex), np.arange(128)
    old = "solve|gfx950|B4|N2^12|R2^7|K2^6|fp64|full"
    oldb = "batched|gfx950|Nmax2^12|NR2^19|S2^0|K2^6|fp64|projected"
    path.write_text(json.dumps({k: dict(opts={"row_groups": 256}, ms_per_iter=1.0) for k in (old, oldb)}))

    def trial(*a, **k):
        raise Trial
    monkeypatch.setattr(autotune, "coordinate_search", trial)
    with pytest.raises(Trial):
        autotune.tune_solve(None, pair, z, rhs)
    with pytest.raises(Trial):
        autotune.tune_batched(None, [dict(pair=pair, z=z, rhs=rhs)], precision="fp64")
    # an entry of these kernels is
    new = {autotune.shape_key(4, 4096, 128, 64, "fp64", "full"): dict(opts={"fuse_steps": 8}, ms_per_iter=1.0)}
    path.write_text(json.dumps(new))
    assert autotune.tune_solve(None, pair, z, rhs) == {"fuse_steps": 8}
