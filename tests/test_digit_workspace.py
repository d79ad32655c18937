"""The workspace a sort by key asks for holds its digit passes at every size: a
key and a payload for each element, and 256 counts for each tile of at most
8,192."""
import pytest

import paper_2409_03970_amd as hv


@pytest.mark.parametrize("n", [1 << 16, 1 << 20, (1 << 22) - 1, 1 << 22, 1 << 24, (1 << 26) - 1,
                               1 << 26, 1 << 28, (1 << 31) - 1])
def test_sort_by_key_workspace_has_room_for_the_digit_passes(n):
    L = hv.lib()
    need = L.hvms_sort_by_key_workspace_bytes(n, None)
    assert need >= 12 * n + (n // 8192) * 1024
    aligned = (4 * n + 255) // 256 * 256
    assert need == aligned + L.hvms_sort_workspace_bytes(n, 1, None)
