"""Settings of emt_sim that the host checks without a device."""
import ctypes as C

import pytest

from paper_1903_01081_amd import _lib, netgen


@pytest.mark.parametrize("value,status", [(0, _lib.EMT_OK), (1, _lib.EMT_OK), (2, _lib.EMT_EINVAL), (-1, _lib.EMT_EINVAL)])
def test_segment_rows_is_zero_or_one(value, status):
    nets = _lib.PackedNets([netgen.small_grid(1, 4)])
    sim = _lib.make_sim(50e-6, 20, 5, segment_rows=value)
    info = _lib.EmtInfo()
    assert _lib.load().emt_analyze(nets.ref, nets.n, C.addressof(sim), C.addressof(info)) == status
