"""The library's host code against a stand-in for the HIP runtime (host_lib.py): no GPU, no kernel runs."""

import numpy as np
import pytest

from host_lib import HostLib, build_host_lib


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return HostLib(build_host_lib(str(tmp_path_factory.mktemp("host_lib"))))


@pytest.mark.parametrize("N,W", [(1, 1), (104096, 64), ((1 << 25) - 1, 1), (1 << 25, 1), (1 << 25, 64), (1 << 25, 65),
                                 ((1 << 25) + 1, 1), (1 << 26, 1), (1 << 28, 1), ((1 << 28) + 1, 1), ((1 << 30) + 1, 1),
                                 (2**31 - 1, 1)])
def test_the_table_of_the_class_grouping_is_cleared_whole(lib, N, W):
    """Slots and lowest members of the table, two words for each of its places, are cleared before ops are put into it, and
    no launch has more threads than a grid can count; what is beyond that is refused (and grouped on the host)."""
    lib.host_forget_launches()
    rc = lib.host_group_rows(N, W)
    if rc != 0:
        assert N > 1 << 25 or N * W > 1 << 31
        assert lib.launches() == []
        return
    slots = 64
    while slots < 2 * N:
        slots *= 2
    assert lib.host_group_bytes(N) >= 48 * N + 8 * slots
    launches = lib.launches()
    assert [l for l in launches if "fill_i32" in l[0]][0][4] == 2 * slots
    for name, blocks, threads, _, filled in launches:
        assert blocks * threads < 1 << 32
        assert blocks * threads >= (filled if "fill_i32" in name else N)
