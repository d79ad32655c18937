"""One captured two-word sort, replayed on inputs whose plans differ: low digits
left out and finished, none left out, constant digits, presorted, reversed, a
second round.  Eager work runs between the replays, and the workspace is
overwritten; in place and not."""
import numpy as np
import pytest
import torch

import paper_2409_03970_amd as hv
from test_gpu_digit_passes import _unsampled

pytestmark = pytest.mark.gpu
DEV = "cuda"
N = (1 << 24) + 4097


def _inputs():
    rng = np.random.default_rng(12)
    wide = rng.integers(-2**63, 2**63, N, dtype=np.int64)
    yield "digits left out", wide
    again = wide.copy()
    at = _unsampled(N, 20000, rng)
    again[at] = (77 << 40) + rng.integers(0, 2**32, len(at))
    yield "second round", again
    yield "presorted", np.sort(wide)
    zeros = np.zeros(N, dtype=np.int64)
    zeros[at[:500]] = rng.integers(1, 1 << 40, 500)
    yield "nearly constant", zeros
    yield "all digits", (wide >> 44) ^ (wide << 44)
    yield "reversed", np.sort(wide)[::-1].copy()
    yield "digits left out again", wide ^ 0x5555


@pytest.mark.parametrize("inplace", (False, True))
@pytest.mark.parametrize("kind", ("i64", "pairs"))
def test_one_graph_for_all_plans(kind, inplace):
    x = torch.zeros(N, dtype=torch.int64, device=DEV)
    k, v = (torch.zeros(N, dtype=torch.int32, device=DEV) for _ in range(2))
    out = x if inplace else torch.empty_like(x)
    ko, vo = (k, v) if inplace else (torch.empty_like(k), torch.empty_like(v))
    L = hv.lib()
    need = (L.hvms_sort64_workspace_bytes(N, None) if kind == "i64"
            else L.hvms_sort_workspace_bytes(N, 1, None))
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())

    def sort():
        if kind == "i64":
            hv.hvms_sort_i64(x, out, ws, stream=s)
        else:
            hv.hvms_sort_pairs_i32(k, v, ko, vo, ws, stream=s)

    with torch.cuda.stream(s):
        sort()
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        sort()
    for what, words in _inputs():
        print("replay", kind, inplace, what, flush=True)
        y = torch.from_numpy(words).to(DEV)
        want = torch.sort(y).values
        x.copy_(y)
        k.copy_(y >> 32)
        v.copy_((y & 0xffffffff) - 2**31)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = out if kind == "i64" else (ko.long() << 32) | (vo.long() + 2**31)
        assert torch.equal(got, want), what
        ws.fill_(0xA5)
