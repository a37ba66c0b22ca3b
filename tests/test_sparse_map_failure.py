"""A sparse map whose upload fails half-way leaves a context from which the exact map can
be restored."""
import ctypes as C

import numpy as np
import pytest

from fake_hip import scenario
from geoms import small


def failed_upload(F, copy):
    og = small()
    h = F.create(og)
    B = np.empty(og.B().shape)
    before = F.rt.fake_memory_hash()
    F.rt.fake_fail_copy(copy)
    rc = F.lib.tt_set_sparse_map(h, 2)
    F.rt.fake_fail_copy(-1)
    F.ok("tt_set_sparse_map", h, 0)
    F.ok("tt_basis_matrix", h, B.ctypes.data_as(C.POINTER(C.c_double)))
    # (the sparse map's own tables are written last)
    return rc, F.rt.fake_memory_hash() == before, float(np.abs(B - og.B()).max())


@pytest.mark.parametrize("copy", [0, 1, 2, 3])
def test_the_exact_map_is_restored(copy):
    rc, restored, error = scenario("test_sparse_map_failure", "failed_upload", copy)
    assert rc == -4 and restored and error < 1e-13
