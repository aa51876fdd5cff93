"""Which leaf launch a call takes (hv_leaf_launch_for), on a device of 256 CUs;
without a GPU."""
import ctypes
import os

import pytest

from paper_2510_23938_amd import hv

CU = 256


def launch(n, alg="sha256", msgs=1, C=65536):
    return hv.leaf_launch_for(msgs, n, C, alg, cus=CU)


@pytest.fixture(autouse=True)
def automatic():
    yield
    hv.set_leaf_kernel("auto")


def test_rule_by_leaf_count():
    for alg, above in (("sha256", "three-group"), ("sha384", "one-wave")):
        assert [launch(n, alg) for n in (1, 64 * CU)] == ["two-wave"] * 2
        assert [launch(n, alg) for n in (64 * CU + 1, 128 * CU)] == ["two-wave-compact"] * 2
        assert [launch(n, alg) for n in (128 * CU + 1, 192 * CU)] == [above] * 2
        assert launch(192 * CU + 1, alg) == "one-wave"
        # just above whole waves per SIMD the work is split evenly, just below it is even
        assert [launch(n, alg) for n in (256 * CU, 512 * CU, 768 * CU)] == ["one-wave"] * 3
        assert [launch(n, alg) for n in (256 * CU + 1, 512 * CU + 64, 768 * CU + 64)] == ["tape"] * 3
        assert launch((1 << 20) + 1, alg) == "one-wave"
        assert launch(256 * CU + 1, alg, C=0) == "one-wave"
        assert launch(256 * CU + 1, alg, msgs=20000) == "one-wave"  # many tails


def test_short_chunks_of_three_groups_per_cu():
    n = 150 * CU
    assert [launch(n, C=C) for C in (128, 256, 512)] == ["one-wave"] * 3
    assert [launch(n, C=C) for C in (576, 1024, 0)] == ["three-group"] * 3


def test_short_chunks_and_many_leaves_keep_the_plain_launch():
    # the tape lost there: three waves on a SIMD, and a launch for its plan
    for alg in ("sha256", "sha384"):
        for n in (256 * CU + 1, 135000, 300000):
            assert [launch(n, alg, C=C) for C in (128, 512, 1024, 1920)] == ["one-wave"] * 4
            assert [launch(n, alg, C=C) for C in (2048, 4096, 16384)] == ["tape"] * 3
            assert [launch(n, alg, msgs=n // 8, C=C) for C in (2048, 4096)] == ["one-wave", "tape"]
        assert [launch(n, alg, C=4096) for n in (450000, 520000, 700000, 1000000)] == ["one-wave"] * 4


def test_a_forced_choice_runs_the_kernel_it_names():
    for n in (100, 128 * CU + 1, 256 * CU + 1, 512 * CU + 64):
        for name in ("one-wave", "two-wave-compact"):
            hv.set_leaf_kernel(name)
            assert launch(n) == launch(n, "sha384") == name
    hv.set_leaf_kernel("two-wave")
    assert [launch(n) for n in (64 * CU, 64 * CU + 1)] == ["two-wave", "two-wave-compact"]


def test_other_devices():
    assert hv.leaf_launch_for(1, 100 * 100, 65536, cus=100) == "two-wave-compact"
    # the tape's scratch is for up to 256 CUs
    assert hv.leaf_launch_for(1, 120000, 65536, cus=304) == "one-wave"


def test_bench_names_the_kernel_that_runs():
    import bench
    csrc = os.path.join(os.path.dirname(os.path.abspath(hv.__file__)), "csrc")
    sources = {}
    for alg in ("sha256", "sha384"):
        sources[alg] = "".join(open(os.path.join(csrc, f"{alg}_{part}.hip")).read() for part in ("leaves", "split"))
    for alg, name in [(a, n) for a in sources for n in ("one-wave", "two-wave", "two-wave-compact", "tape")] + \
            [("sha256", "three-group")]:
        assert f" {bench.leaf_kernel_name(alg, name)}(" in sources[alg]


def test_errors():
    k = ctypes.c_int(0)
    assert hv.lib.hv_leaf_launch_for(7, 1, 10, 4096, CU, ctypes.byref(k)) == hv.HV_ERR_INVALID_ARG
    assert hv.lib.hv_leaf_launch_for(0, 1, 10, 4096, CU, None) == hv.HV_ERR_INVALID_ARG
