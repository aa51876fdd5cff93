"""Message tables packed by the library against numpy's, around the counts from
which the binding has them filled by it and from which several threads fill
them; without a GPU."""
import numpy as np
import pytest

from paper_2510_23938_amd import hv


@pytest.mark.parametrize("n", [0, 1, 3, (1 << 16) + 17, hv._PACK_MIN - 1, hv._PACK_MIN, hv._PACK_MIN + 17])
@pytest.mark.parametrize("dtype,step", [(np.uint64, 1), (np.int64, 1), (np.uint64, 2)])
def test_pack(n, dtype, step):
    rng = np.random.default_rng(n)
    ptrs = rng.integers(0, 1 << 62, n * step).astype(dtype)[::step]
    lens = rng.integers(0, 1 << 40, n * step).astype(dtype)[::step]
    host = hv.HostBuffer(pinned=False)
    want = np.stack([ptrs.astype(np.uint64), lens.astype(np.uint64)], axis=1)
    assert np.array_equal(hv._packed_msgs(ptrs, lens), want)
    assert np.array_equal(hv._packed_msgs(ptrs, lens, host), want)


@pytest.mark.parametrize("n", [1, (1 << 16) + 17, (1 << 19) - 1, (1 << 19) + 17])
def test_library(n):
    rng = np.random.default_rng(n)
    ptrs, lens = rng.integers(0, 1 << 62, n, dtype=np.uint64), rng.integers(0, 1 << 40, n, dtype=np.uint64)
    got = np.zeros((n, 2), dtype=np.uint64)
    assert hv.lib.hv_pack_messages(ptrs.ctypes.data, lens.ctypes.data, n, got.ctypes.data) == hv.HV_OK
    assert np.array_equal(got, np.stack([ptrs, lens], axis=1))


def test_who_packs(monkeypatch):
    """Small tables, and arrays that are no aligned rows of 64-bit words, are left to numpy."""
    calls = []
    monkeypatch.setattr(hv.lib, "hv_pack_messages", lambda *a: calls.append(a) or 0)
    a = np.zeros(hv._PACK_MIN, dtype=np.uint64)
    odd = np.frombuffer(bytes(8 * len(a) + 1), dtype=np.uint8)[1:].view(np.uint64)
    assert not odd.flags.aligned
    for ptrs, lens in [(a[1:], a[1:]), (odd, a), (a, odd), (a.astype(np.int64), a), (a, a.reshape(1, -1)[0][::-1])]:
        hv._packed_msgs(ptrs, lens)
    assert not calls
    hv._packed_msgs(a, a)
    assert len(calls) == 1


def test_errors():
    a = np.zeros(4, dtype=np.uint64)
    assert hv.lib.hv_pack_messages(a.ctypes.data, None, 2, a.ctypes.data) == hv.HV_ERR_INVALID_ARG
    assert hv.lib.hv_pack_messages(None, None, 0, None) == hv.HV_OK
    with pytest.raises(ValueError):
        hv._packed_msgs(np.zeros(3, np.uint64), np.zeros(2, np.uint64))
