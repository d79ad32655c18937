"""The workspace of the CDF model's training holds a row of 1,154 partial sums for
each workgroup (128 samples, at most 256 workgroups) and nothing else."""
import os

import pytest

import paper_2409_03970_amd as hv

pytestmark = pytest.mark.skipif(not os.path.exists(hv.LIB_PATH), reason="libhvms.so not built")


@pytest.mark.parametrize("b", [1, 127, 128, 129, 4096, 32767, 32768, 32769, 65536, 1 << 20,
                               (1 << 62) + 1])
def test_training_workspace_is_the_rows_of_partials(b):
    L = hv.lib()
    rows = min(256, -(-b // 128))
    need = -(-rows * 1154 * 4 // 256) * 256
    assert b > 1 << 40 or L.hvms_cdf_workspace_bytes(b) >= need
    assert L.hvms_cdf_train_workspace_bytes(b) == need


def test_no_samples():
    L = hv.lib()
    assert L.hvms_cdf_workspace_bytes(0) == 0 and L.hvms_cdf_workspace_bytes(-1) == -1
    assert L.hvms_cdf_train_workspace_bytes(0) == L.hvms_cdf_train_workspace_bytes(-1) == -1
