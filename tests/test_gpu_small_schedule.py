"""The one-launch scheduler of calls of few messages and the launches of larger
ones, at the message counts around a wave (64) and their boundary (1024):
every chunk once with its source range and leaf number, longest class first,
and listed chunks rehashed where they belong."""
import numpy as np
import pytest
import torch

from paper_2510_23938_amd import hv
from test_gpu_schedule import blocks, expected_leaves, sort_class

pytestmark = pytest.mark.gpu
COUNTS = [1, 2, 63, 64, 65, 1023, 1024, 1025]


def messages(n, seed):
    """Lengths with empty messages, whole chunks only and single tails among them, back to back."""
    rng = np.random.default_rng([n, seed])
    lens = rng.integers(0, 3000, n)
    lens[rng.random(n) < 0.2] = 0
    whole = rng.random(n) < 0.2
    lens[whole] = lens[whole] // 128 * 128
    lens[rng.integers(0, n)] = 400000 + int(rng.integers(0, 500))
    buf = torch.zeros(int(lens.sum()) + 16, dtype=torch.uint8, device="cuda").random_(0, 256)
    starts = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.uint64)
    return buf, np.uint64(buf.data_ptr()) + starts, lens.astype(np.uint64)


@pytest.mark.parametrize("C", [128, 1024, 0])
@pytest.mark.parametrize("n", COUNTS)
def test_schedule(n, C):
    buf, ptrs, lens = messages(n, C)
    table = hv.hv_leaf_schedule((ptrs, lens), C)
    got = sorted(tuple(int(x) for x in r) for r in table)
    assert got == sorted(expected_leaves(ptrs, lens, C))
    key = [sort_class(blocks(int(r[1]))) for r in table]
    assert all(a >= b for a, b in zip(key, key[1:])), "not longest-first"


@pytest.mark.parametrize("C", [128, 0])
@pytest.mark.parametrize("n", COUNTS)
def test_rehash(n, C):
    buf, ptrs, lens = messages(n, C + 1)
    want, _ = hv.hv_hash_chunks((ptrs, lens), C)
    k = want.shape[0]
    rng = np.random.default_rng(n)
    listed = np.unique(np.concatenate([[0, k - 1], rng.integers(0, k, min(k, 1500))])).astype(np.uint64)
    got = torch.zeros_like(want)
    hv.hv_rehash_chunks((ptrs, lens), C, listed, got)
    at = torch.from_numpy(listed.astype(np.int64)).cuda()
    assert torch.equal(got[at], want[at])
    others = torch.ones(k, dtype=torch.bool, device="cuda")
    others[at] = False
    assert not got[others].any()


# Tables that fill a launch's arguments (480 words, 960 where they fit 32 bits)
# or all four launches', and one message or leaf more.
@pytest.mark.parametrize("n,k", [(240, 960), (241, 961), (960, 3840), (961, 3841), (1440, 5760), (1441, 5761)])
def test_tables_in_arguments(n, k):
    lens = np.full(n, 128 * 6, dtype=np.uint64)
    buf = torch.zeros(int(lens.sum()), dtype=torch.uint8, device="cuda").random_(0, 256)
    ptrs = np.uint64(buf.data_ptr()) + np.arange(n, dtype=np.uint64) * np.uint64(128 * 6)
    want, seg = hv.hv_hash_chunks((ptrs, lens), 128)
    leaves = np.sort(np.random.default_rng(n).choice(6 * n, k, replace=False)).astype(np.uint64)
    at = torch.from_numpy(leaves.astype(np.int64)).cuda()
    got = want.clone()
    got[at] = 0
    tree = hv.Tree(got, seg)
    hv.hv_rehash_chunks((ptrs, lens), 128, leaves, got)
    roots = tree.update(got, leaves)
    assert torch.equal(got, want)
    assert torch.equal(roots, hv.hv_merkle_reduce(want, seg))
