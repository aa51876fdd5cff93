"""The one-wave leaf kernels over a tape: the leaf table's work cut into one
equal interval per resident wave, chunks across a boundary hashed by two waves.

Leaf counts just above one, two, three and four waves per SIMD, where an
interval is about one chunk long and every chunk is cut, and counts whose last
group is partly filled; tails from none to one leaf in four (and to more than
256 groups of them, several per thread of the plan), tails of every length below
a chunk, and chunks at and above the block count (2048) where the scheduler's
classes stop being exact, so that a group's tape length is only a bound.  Every
case says that it runs on a tape.  Digests are bytes, compared with hashlib's
for every leaf.
"""
import concurrent.futures as futures
import hashlib

import numpy as np
import pytest
import torch

import workloads as W

from paper_2510_23938_amd import hv  # noqa: E402  (a missing library fails the run, never skips it)

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda")


def expected(host, starts, lens, C, alg):
    H = getattr(hashlib, alg)

    def message(i):
        s, n = int(starts[i]), int(lens[i])
        return b"".join(H(host[s + o:s + min(o + C, n)]).digest() for o in range(0, n, C))

    with futures.ThreadPoolExecutor(8) as pool:
        return b"".join(pool.map(message, range(len(lens))))


# (leaves, chunk, messages, all but one of them with a tail, the bytes past 16
# they start at)
CASES = [
    (65536 + 1, 2048, 1, 0), (65536 + 100, 2176, 4, 0), (70001, 4096, 66, 3), (98304, 2304, 1000, 0),
    (131072 + 63, 2048, 70, 0), (196608 + 64, 2048, 700, 1), (66000, 4096, 16500, 0), (70000, 4224, 17500, 5),
    (270000, 4096, 60000, 0),
]


@pytest.mark.parametrize("alg", ["sha256", "sha384"])
@pytest.mark.parametrize("n,C,count,shift", CASES)
def test_digests(alg, n, C, count, shift):
    assert hv.leaf_launch_for(count, n, C, alg) == "tape"
    rng = np.random.default_rng(n + C)
    tails = count - 1
    whole = rng.multinomial(n - tails, np.full(count, 1 / count)) * C
    lens = rng.permutation(whole + np.concatenate(([0], rng.integers(1, C, tails))))
    starts = shift + np.concatenate(([0], np.cumsum((lens + 15) // 16 * 16)[:-1]))
    buf = W.random_bytes(int(starts[-1] + lens[-1]), 7, DEV)
    table = hv._msg_array(np.uint64(buf.data_ptr()) + starts.astype(np.uint64), lens)
    _, leaves = hv._layout_of(table, C)
    assert leaves == n
    got, _ = hv.hv_hash_chunks((table[:, 0], table[:, 1]), C, alg=alg)
    assert got.cpu().numpy().tobytes() == expected(buf.cpu().numpy(), starts, lens, C, alg)


@pytest.mark.parametrize("alg", ["sha256", "sha384"])
def test_long_chunks_and_inexact_classes(alg):
    # 192 KiB chunks (3072 blocks) and tails around 2048 blocks, in one buffer
    # read by every message: the digests repeat, the work does not
    C, n = 192 << 10, 65536 + 128
    buf = W.random_bytes(C, 8, DEV)
    tails = np.arange(1000) * 61 + 100000
    # messages of 8 chunks, so that they are few per leaf
    eight = buf.repeat(8)
    whole = (n - len(tails)) // 8
    assert hv.leaf_launch_for(whole + len(tails), n, C, alg) == "tape"
    ptrs = np.concatenate((np.full(whole, eight.data_ptr()), np.full(len(tails), buf.data_ptr()))).astype(np.uint64)
    lens = np.concatenate((np.full(whole, 8 * C), tails)).astype(np.uint64)
    got, _ = hv.hv_hash_chunks((ptrs, lens), C, alg=alg)
    got = got.cpu().numpy()
    host = buf.cpu().numpy().tobytes()
    H = getattr(hashlib, alg)
    assert (got[:8 * whole] == np.frombuffer(H(host).digest(), dtype=np.uint8)).all()
    for i, t in enumerate(tails):
        assert got[8 * whole + i].tobytes() == H(host[:int(t)]).digest()


@pytest.mark.parametrize("alg", ["sha256", "sha384"])
def test_a_wave_that_gives_up_hashes_the_chunks_itself(alg):
    # no look for the other wave's states: every cut group is hashed from its
    # first block by the wave that ends it
    n, C = 65536 + 700, 4096
    assert hv.leaf_launch_for(1, n, C, alg) == "tape"
    buf = W.random_bytes(n * C - 77, 10, DEV)
    msgs = (np.array([buf.data_ptr() + 1], dtype=np.uint64), np.array([n * C - 78], dtype=np.uint64))
    want, _ = hv.hv_hash_chunks(msgs, C, alg=alg)
    assert want.cpu().numpy().tobytes() == expected(buf.cpu().numpy(), [1], [n * C - 78], C, alg)
    hv.lib.hv_set_handover_polls(0)
    try:
        got, _ = hv.hv_hash_chunks(msgs, C, out=torch.zeros_like(want), alg=alg)
        torch.cuda.synchronize()
    finally:
        hv.lib.hv_set_handover_polls(1 << 14)
    assert torch.equal(got, want)


def test_workspace_without_tape_and_repeated_runs():
    n, C = 70000, 4096
    assert hv.leaf_launch_for(1, n, C) == "tape"
    buf = W.random_bytes(n * C - 5, 9, DEV)
    msgs = (np.array([buf.data_ptr()], dtype=np.uint64), np.array([n * C - 5], dtype=np.uint64))
    want, _ = hv.hv_hash_chunks(msgs, C)
    assert want.cpu().numpy().tobytes() == expected(buf.cpu().numpy(), [0], [n * C - 5], C, "sha256")
    # the table's own bytes are workspace enough; the plain launch then runs
    full = hv.lib.hv_hash_workspace_bytes(1, n)
    table = hv._msg_array(*msgs)
    small = torch.empty(full - (12 << 20), dtype=torch.uint8, device=DEV)
    out = torch.zeros_like(want)
    assert hv.lib.hv_hash_chunks(table.ctypes.data, 1, C, out.data_ptr(), small.data_ptr(), small.numel(),
                                 hv._stream(DEV)) == hv.HV_OK
    assert torch.equal(out, want)
    # a prepared pass, run and replayed: the hand-over flags are cleared each time
    pipe = hv.Pipeline(msgs, C)
    root = bytes(pipe.compute().cpu().numpy().reshape(-1))
    pipe.capture(root)
    for k in range(3):
        buf[k] ^= 1
        assert not pipe.replay() and not pipe.run(root)
        buf[k] ^= 1
        assert pipe.replay() and pipe.run(root)
    assert torch.equal(pipe.leaves, want)
