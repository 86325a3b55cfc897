"""Cache entries of the autotuner that were saved before a ring had transform
kernels: they named int8 row passes and are not applied any more; where the
kernels are the same as then, they still are."""
import json

import pytest

import seeded_inputs as si
from paper_2510_15413_amd import autotune

OLD = {"max_batch": 32, "row_pass": 8, "split_groups": -1}
NEW = {"max_batch": 64, "row_pass": 0, "split_groups": -1}


class Ctx:
    def __init__(self, p):
        self.p, self.applied = p, []

    def set_tuning(self, **kw):
        self.applied.append(kw)


@pytest.mark.parametrize("q,N,stale", [(32, 1024, True), (32, 2048, True), (64, 1024, True), (64, 2048, True),
                                       (32, 256, True), (32, 512, False), (64, 512, False), (64, 256, False),
                                       (32, 64, False)])
def test_entries_of_the_int8_kernels(tmp_path, monkeypatch, q, N, stale):
    monkeypatch.setattr(autotune, "_gpu_name", lambda: "gpu")
    p = si.Params("old", q, 630, 1, N, 7, 3, 2, 8, 15, 25)
    cache = tmp_path / "tune.json"
    old_key = f"gpu|q{q} n630 N{N} l3 bg7 ks2x8|load"
    cache.write_text(json.dumps({old_key: {"best": OLD, "times": []}}))
    ran = []
    ctx = Ctx(p)
    best, _ = autotune.tune(ctx, "load", lambda: ran.append(1), cands=[NEW], cache_path=str(cache))
    assert best == (NEW if stale else OLD) and ctx.applied[-1] == best and bool(ran) == stale
    again = Ctx(p)
    assert autotune.tune(again, "load", lambda: 1 / 0, cands=[NEW], cache_path=str(cache))[0] == best
    assert json.loads(cache.read_text())[old_key]["best"] == OLD
