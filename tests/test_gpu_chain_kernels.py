"""The two-lane chain kernels at their edges against the CPU oracle: chunk
counts around a consumer wave (32) and a group (64), block counts around the
three schedule buffers and the two alternate producers, chunks that end blocks
before their neighbours, and every start within a 16-byte granule.  Digests are
compared exactly."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle

from paper_2510_23938_amd import hv

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda")
BLOCK = {"sha256": 64, "sha384": 128}


def run_lengths(lens, align, alg, seed):
    """Leaf digests of whole messages of these lengths, message i starting ``align`` * i mod 16 past a granule."""
    starts, pos = [], 0
    for i, n in enumerate(lens):
        starts.append(pos + align * i % 16)
        pos = (starts[-1] + n + 31) // 16 * 16
    buf = W.random_bytes(pos + 16, seed, DEV)
    ptrs = np.uint64(buf.data_ptr()) + np.array(starts, dtype=np.uint64)
    leaves, _ = hv.hv_hash_chunks((ptrs, np.array(lens, dtype=np.uint64)), 0, alg=alg)
    host = buf.cpu().numpy()
    want = oracle.leaf_digests_mt([host[s:s + n].tobytes() for s, n in zip(starts, lens)], 0, 4, alg)
    return leaves.cpu().numpy(), want


@pytest.mark.parametrize("alg", ["sha256", "sha384"])
@pytest.mark.parametrize("align", [0, 1])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 127, 129])
def test_edges(n, align, alg):
    hv.set_leaf_kernel("two-wave")
    try:
        for blocks in range(1, 9):  # the group's most blocks, padding included
            top = blocks * BLOCK[alg] - (9 if alg == "sha256" else 17)
            rng = np.random.default_rng([n, blocks])
            lens = rng.integers(0, top, n, endpoint=True)
            lens[rng.integers(0, n)] = top
            got, want = run_lengths([int(x) for x in lens], align, alg, 900 + blocks)
            assert np.array_equal(got, want), f"{blocks} blocks"
    finally:
        hv.set_leaf_kernel("auto")


@pytest.mark.parametrize("alg", ["sha256", "sha384"])
@pytest.mark.parametrize("choice", ["one-wave", "two-wave", "two-wave-compact"])
def test_no_bytes_at_odd_addresses(choice, alg):
    # blocks that hold none of a chunk's bytes (an empty message's, and the
    # length-only one after a long tail) are formed without loads
    hv.set_leaf_kernel(choice)
    try:
        tail = BLOCK[alg] - 1
        got, want = run_lengths([0, tail, 0, BLOCK[alg] + tail, BLOCK[alg], 0, 1], 5, alg, 31)
        assert np.array_equal(got, want)
    finally:
        hv.set_leaf_kernel("auto")


@pytest.mark.parametrize("align", [0, 1])
@pytest.mark.parametrize("per_cu", [128, 150, 192])
def test_three_groups_per_cu(per_cu, align):
    # above 128 and up to 192 chunks per CU: workgroups (the table is sorted by
    # length) whose longest chunk has 1 to 12 blocks and one of 70, the last
    # workgroup partly filled
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = per_cu * cus + (1 if per_cu == 128 else 0)
    assert hv.leaf_launch_for(n, n, 0) == "three-group"
    rng = np.random.default_rng([per_cu, align])
    lens = rng.integers(0, 12 * 64 - 9, n, endpoint=True)
    lens[rng.integers(0, n, 5)] = 70 * 64 - 9
    got, want = run_lengths([int(x) for x in lens], align, "sha256", 950)
    assert np.array_equal(got, want)
