"""The allocation-free sort at the sizes where its fixed scratch holds the counts
of 8,192-key tiles only, and at the edges of that range, twice on one scratch."""
import pytest
import torch

import paper_2409_03970_amd as hv
from paper_2409_03970_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", [3_840_000, 3_850_241, 8192 * 489, 8192 * 489 + 1, (1 << 22) - 1,
                               1 << 22])
def test_noalloc_sizes(n):
    for dist in ("zipf", "uniform", "reverse", "sorted"):
        print("noalloc", n, dist, flush=True)
        x = inputs.keys(n, dist, seed=n, device=DEV) - (1 << 30)
        y = torch.full_like(x, -1)
        hv.hvms_sort_i32_noalloc(x, y)
        assert torch.equal(y, torch.sort(x).values)
        hv.hvms_sort_i32_noalloc(x, x)
        assert torch.equal(x, y)
