"""Reductions of many short segments: group launches in place of a tile per segment."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle

from paper_2510_23938_amd import hv  # noqa: E402  (a missing library fails the run, never skips it)


def offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)


def kinds(sizes, alg="sha256"):
    return [p[0] for p in hv.merkle_launches(offsets(sizes), alg, cus=256)]


def test_launch_plan():
    assert kinds([5] * 1536) == ["tile"]
    assert kinds([5] * 1537) == ["group"]
    assert kinds([8] * 1537) == ["group"] and kinds([9] * 1537) == ["tile"]  # up to 8 entries on average
    assert kinds([0] * 1537) == ["group"]
    assert kinds([5] * 2000 + [9]) == ["group", "group"]
    # a long segment among short ones: as many group launches as save a tile
    # launch, tiles where none would be saved
    assert kinds([2] * 3100 + [4000]) == ["group", "tile"]
    assert kinds([2] * 3100 + [12000]) == ["group", "group", "tile"]
    assert kinds([5] * 3073 + [500]) == ["group"] * 3 and kinds([5] * 3071 + [500]) == ["tile"]
    assert kinds([2] * 2000 + [4000]) == ["tile", "group"] and kinds([2] * 2000 + [12000]) == ["tile", "tile"]
    assert kinds([5] * 20000 + [300000]) == ["group", "tile", "tile"]
    assert kinds([8] * 60000 + [12000]) == kinds([9] * 60000 + [12000]) == ["group", "group", "tile"]
    assert kinds([40] * 60000 + [12000]) == ["group", "group", "tile"]
    assert kinds([10] * 60000) == ["group", "group"]
    # or where many nodes each are left to the tiles
    assert kinds([40] * 20000 + [300000]) == ["group", "group", "tile", "tile"]
    # nor where the tiles are as quick
    assert kinds([2] * 3072, "sha384") == ["tile"] and kinds([2] * 3073, "sha384") == ["group"]
    assert kinds([3] * 1537, "sha384") == ["group"]
    # no deeper a chain than without the rule
    assert len(kinds([1] * 200000 + [1 << 21])) <= 8
    # four lanes a group up to two rounds of them
    assert hv.merkle_launches(offsets([5] * 20000), cus=256) == [("group", 20000, 0)]
    assert hv.merkle_launches(offsets([5] * 32769), cus=256) == [("group", 32769, 32769)]
    # a workspace for more entries always holds fewer
    need = [hv.lib.hv_merkle_workspace_bytes(n, 2000) for n in range(0, 1 << 19, 997)]
    assert need == sorted(need)


@pytest.mark.gpu
@pytest.mark.parametrize("alg", ["sha256", "sha384"])
@pytest.mark.parametrize("sizes", [
    [k % 9 for k in range(1537)],                 # every group size, empty ones too, four lanes each
    [k % 14 for k in range(33000)],               # one lane each, two launches
    [1 + k % 3 for k in range(3100)] + [4000, 0, 513],
    [1 + k % 3 for k in range(3100)] + [500, 0, 512],
], ids=["four_lanes", "one_lane", "one_long", "three_launches"])
def test_roots(alg, sizes):
    D = 32 if alg == "sha256" else 48
    seg = offsets(sizes)
    assert hv.merkle_launches(seg, alg)[0][0] == "group"
    n = int(seg[-1])
    entries = W.random_bytes(n * D, 400 + D, torch.device("cuda")).view(n, D)
    roots = hv.hv_merkle_reduce(entries, seg, alg=alg).cpu().numpy()
    host = entries.cpu().numpy()
    assert [bytes(r) for r in roots] == \
        [oracle.mth(host[int(seg[k]):int(seg[k + 1])], alg) for k in range(len(sizes))]
