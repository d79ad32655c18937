"""The workspace a sort by key asks for holds its digit passes at every size: a
key and a payload for each element, and 256 counts for each tile (8,192 keys at
most, 16,384 from 2^25 keys on)."""
import pytest

import paper_2409_03970_amd as hv


@pytest.mark.parametrize("n", [1 << 16, 1 << 20, (1 << 22) - 1, 1 << 22, 1 << 24, (1 << 25) - 1,
                               1 << 25, (1 << 26) - 1, 1 << 26, 1 << 28, (1 << 31) - 1])
def test_sort_by_key_workspace_has_room_for_the_digit_passes(n):
    L = hv.lib()
    need = L.hvms_sort_by_key_workspace_bytes(n, None)
    tile = 8192 if n < 1 << 25 else 16384
    assert need >= 12 * n + (n // tile) * 1024
    aligned = (4 * n + 255) // 256 * 256
    assert need == aligned + L.hvms_sort_workspace_bytes(n, 1, None)
