"""Keys of the tuning cache that are not this package's are passed over, and the
options handed out are the caller's own."""
import json

import torch

from paper_2409_03970_amd import tune


def test_foreign_keys_are_passed_over(tmp_path):
    p = str(tmp_path / "cache.json")
    good = {"options": {"merge_ways": 2}}
    with open(p, "w") as f:
        json.dump({"a:b:c:x": 1, "a:b:c:": {}, "a:b:c:-3": [], "a:b:c:2.5": {}, "gfx950:256:sort:20":
                   good, "x": {}, "a:b:c:d:1": {}}, f)
    assert tune._entries(p) == (("gfx950:256:sort", 20, good),)


def test_options_handed_out_are_copies(tmp_path, monkeypatch):
    p = str(tmp_path / "cache.json")
    with open(p, "w") as f:
        json.dump({"gfx950:256:sort:20": {"options": {"merge_ways": 4}}}, f)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(tune, "_key", lambda op, log2n: f"gfx950:256:{op}:{log2n}")
    o = tune.tuned_options("sort", 1 << 20, path=p)
    o["merge_ways"] = 2
    assert tune.tuned_options("sort", 1 << 20, path=p) == {"merge_ways": 4}
