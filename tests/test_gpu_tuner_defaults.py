"""What the tuner records for a plain sort is a merge shape, the defaults among
them: an entry with no option set would stand for the digit passes."""
import json

import pytest

import paper_2409_03970_amd as hv
from paper_2409_03970_amd import tune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op,log2n", (("sort", 18), ("sort_pairs", 22)))
def test_recorded_shapes_are_merge_shapes(op, log2n, tmp_path):
    p = str(tmp_path / "cache.json")
    four = dict(keys_per_lane=16, block_threads=512, merge_tile=4096, merge_ways=4)
    tune.tune(op, log2n, reps=1, path=p, cands=[four], verbose=False)
    (entry,) = json.load(open(p)).values()
    assert entry["options"] in (four, {"merge_ways": 2})
    assert entry["two_way"]["options"] == {"merge_ways": 2}
    n, pairs = 1 << log2n, int(op == "sort_pairs")
    # and it runs in a workspace of the merge sort's size
    L = hv.lib()
    assert (L.hvms_sort_workspace_bytes(n, pairs, hv._opts(entry["two_way"]["options"]))
            < L.hvms_sort_workspace_bytes(n, pairs, None))
