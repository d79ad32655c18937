"""Groups that the top digits leave alike, at the lengths where the finish hands
them on: a window's lanes, a wave (64 and 256), a tile, two merged tiles, the
longest and more than the list holds.  They are planted where the sample does
not look, half of them with few different elements."""
import numpy as np
import pytest
import torch

import paper_2409_03970_amd as hv
from test_gpu_digit_passes import _unsampled

pytestmark = pytest.mark.gpu
DEV = "cuda"
LENGTHS = [(63, 64, 65, 66, 95, 96, 97, 127, 128, 129) * 9, (191, 192, 193, 255, 256, 257, 258) * 9,
           (8191, 8192, 8193, 8194, 12288), (16383, 16384), (16385,), (16384, 16640, 16641),
           (34,) * 65537, (48,) * 131073]


@pytest.mark.parametrize("inplace", (False, True))
@pytest.mark.parametrize("kind", ("i64", "pairs"))
@pytest.mark.parametrize("lengths", LENGTHS, ids=lambda t: f"{len(t)}x{t[0]}")
def test_listed_groups(lengths, kind, inplace):
    n = (1 << 24) + 4099
    print("listed groups", kind, lengths[:5], len(lengths), inplace, flush=True)
    rng = np.random.default_rng(len(lengths) + lengths[0])
    x = rng.integers(-2**63, 2**63, n, dtype=np.int64)
    at = _unsampled(n, sum(lengths), rng)
    x[at] = np.repeat(rng.integers(-2**31, 2**31, len(lengths), dtype=np.int64) << 32, lengths)
    few = np.repeat(np.arange(len(lengths)) % 2 == 1, lengths)
    x[at] += np.where(few, rng.integers(0, 3, len(at)) * 77777777, rng.integers(0, 2**32, len(at)))
    x = torch.from_numpy(x).to(DEV)
    want = torch.sort(x).values
    if kind == "i64":
        out = x if inplace else torch.empty_like(x)
        assert torch.equal(hv.sort_keys(x, out=out), want)
        return
    k, v = (x >> 32).int(), ((x & 0xffffffff) - 2**31).int()
    ko, vo = (k, v) if inplace else (None, None)
    ko, vo = hv.sort_pairs(k, v, ko, vo)
    assert torch.equal((ko.long() << 32) | (vo.long() + 2**31), want)
