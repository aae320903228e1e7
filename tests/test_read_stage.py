"""Where the staging of a field read-out comes from: device memory, less of it where the device has
less room, and host memory where it has none, so that a full device can still be read."""
import numpy as np
import pytest

import _host_plan as H

ROW = 2000 * 8


@pytest.mark.parametrize("room,bytes_", [(1 << 40, 200 * ROW), (200 * ROW, 200 * ROW), (200 * ROW - 1, 100 * ROW),
                                         (ROW, ROW), (2 * ROW, 25 * ROW // 16)])
def test_device_memory_while_there_is_room(room, bytes_):
    assert H.stage(room, False, 200 * ROW, ROW) == (0, bytes_, False, "device")


@pytest.mark.parametrize("room", [0, ROW - 1])
def test_host_memory_for_a_full_device(room):
    assert H.stage(room, True, 200 * ROW, ROW) == (0, 200 * ROW, True, "host")


def test_neither():
    e, bytes_, _, where = H.stage(0, False, 200 * ROW, ROW)
    assert e != 0 and bytes_ == 0 and where == "none"


@pytest.mark.gpu
@pytest.mark.parametrize("which", [0, 1, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16_neq"])
def test_same_field_through_either(precision, which):
    a, b = (H.field_through(301, 37, precision, which, host) for host in (False, True))
    assert np.isfinite(a).all() and (which != 1 or a.any())
    np.testing.assert_array_equal(a, b)
