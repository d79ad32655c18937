"""The tuning cache is parsed once per state of its file."""
import json
import os

from paper_2409_03970_amd import tune


def test_entries_follow_the_file(tmp_path):
    p = str(tmp_path / "cache.json")
    assert tune._entries(p) == ()
    with open(p, "w") as f:
        json.dump({"gfx950:256:sort:20": {"options": {"merge_ways": 2}}, "odd": {}}, f)
    assert tune._entries(p) == (("gfx950:256:sort", 20, {"options": {"merge_ways": 2}}),)
    assert tune._entries(p) is tune._entries(p)
    with open(p + ".new", "w") as f:
        json.dump({"gfx950:256:sort:21": {"options": {"merge_ways": 4}}}, f)
    os.replace(p + ".new", p)
    assert tune._entries(p) == (("gfx950:256:sort", 21, {"options": {"merge_ways": 4}}),)
    assert [e[0] for e in tune._entries(tune.CACHE)]      # another path
    assert tune._entries(p)[0][1] == 21
