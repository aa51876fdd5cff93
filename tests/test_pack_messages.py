"""Message tables packed by the library against numpy's, around the count from
which several threads fill them; without a GPU."""
import numpy as np
import pytest

from paper_2510_23938_amd import hv


@pytest.mark.parametrize("n", [0, 1, 3, (1 << 16) - 1, 1 << 16, (1 << 16) + 17])
@pytest.mark.parametrize("dtype,step", [(np.uint64, 1), (np.int64, 1), (np.uint64, 2)])
def test_pack(n, dtype, step):
    rng = np.random.default_rng(n)
    ptrs = rng.integers(0, 1 << 62, n * step).astype(dtype)[::step]
    lens = rng.integers(0, 1 << 40, n * step).astype(dtype)[::step]
    host = hv.HostBuffer(pinned=False)
    want = np.stack([ptrs.astype(np.uint64), lens.astype(np.uint64)], axis=1)
    assert np.array_equal(hv._packed_msgs(ptrs, lens), want)
    assert np.array_equal(hv._packed_msgs(ptrs, lens, host), want)


def test_errors():
    a = np.zeros(4, dtype=np.uint64)
    assert hv.lib.hv_pack_messages(a.ctypes.data, None, 2, a.ctypes.data) == hv.HV_ERR_INVALID_ARG
    assert hv.lib.hv_pack_messages(None, None, 0, None) == hv.HV_OK
    with pytest.raises(ValueError):
        hv._packed_msgs(np.zeros(3, np.uint64), np.zeros(2, np.uint64))
