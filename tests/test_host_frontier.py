"""Host side of the frontier form of TAC, against the stand-in for the HIP runtime: which calls take it, memory that runs out
while its tables are made, and streams under capture."""

import numpy as np
import pytest

from paper_1803_03288_amd import workloads as wl

from test_gpu_tac_frontier import GRAPHS as LISTS
from test_host import GRAPHS, layered, lib          # noqa: F401  (lib: the fixture)

LARGE = 600                                         # samples: more than two per compute unit


def names(lib):
    return [n for n in ("tac_frontier_kernel", "tac_sliced_kernel", "tac_kernel") if any(n in k for k in lib.kernels())]


def tac(lib, h, d, B, rc=0):
    lib.host_forget_launches()
    assert lib.tac(h, d, B) == rc, lib.error()
    return names(lib)


@pytest.mark.parametrize("B,frontier", [(1, False), (512, False), (513, True), (LARGE, True)])
def test_batches_that_take_the_frontier_form(lib, B, frontier):
    d = GRAPHS["wide"]()
    h = lib.build(d)[1]
    assert tac(lib, h, d, B) == ["tac_frontier_kernel"] * frontier + ["tac_sliced_kernel", "tac_kernel"]
    lib.free(h)


@pytest.mark.parametrize("name,frontier", [("q127", True), ("q140", True), ("q200", False), ("frontier300", True), ("frontier500", True),
                                           ("frontier400", False), ("frontier900", False), ("in64", True), ("in65", False),
                                           ("wide260", True), ("wide400", False)])
def test_graphs_whose_samples_outgrow_the_lists(lib, name, frontier):
    """(And classes with more inputs than the form takes.)  Where every sample would be left to the bit-sliced kernel, that takes the batch at once; a little beyond the lists'
    lengths samples may fit or not."""
    d = layered(40, int(name[4:]), 800) if name.startswith("wide") else LISTS[name]()
    h = lib.build(d)[1]
    assert tac(lib, h, d, LARGE) == ["tac_frontier_kernel"] * frontier + ["tac_sliced_kernel", "tac_kernel"]
    lib.free(h)


def test_under_capture(lib):
    """A first call allocates, which the runtime refuses under capture; a later one is launches only."""
    d = GRAPHS["wide"]()
    h = lib.build(d)[1]
    lib.tictac_trim_memory()
    lib.host_capturing(1)
    rc = lib.tac(h, d, LARGE)
    lib.host_capturing(0)
    lib.hipGetLastError()
    assert rc == -7
    want = tac(lib, h, d, LARGE)
    assert "tac_frontier_kernel" in want
    waits = lib.count("waits")
    lib.host_capturing(1)
    again = tac(lib, h, d, LARGE)
    lib.host_capturing(0)
    assert again == want and lib.count("waits") == waits
    lib.free(h)


# the second: large enough that the frontier form's tables are planned by a thread of their own
@pytest.mark.parametrize("levels,width", [(12, 160), (20, 300)])
def test_memory_that_runs_out(lib, levels, width):
    """Every allocation of device and of host memory that a first call makes fails once, one after the other: the call makes do
    without or says so, and the next one is as on a fresh handle."""
    d = layered(levels, width, 300)
    assert (d.n_ops + d.row_ptr[-1] > 16384) == (levels == 20)
    h = lib.build(d)[1]
    want = tac(lib, h, d, LARGE)
    assert "tac_frontier_kernel" in want
    lib.free(h)
    for order, left in ((lib.host_fail_device, lib.host_fail_device_left), (lib.host_fail_new, lib.host_fail_new_left)):
        for k in range(4000):
            h = lib.build(d)[1]
            assert lib.tictac_trim_memory() == 0
            order(k)
            rc = lib.tac(h, d, LARGE)
            struck = left() < 0
            order(-1)
            assert rc in (0, -7, -8), (k, lib.error())
            assert lib.hipGetLastError() == 0, k
            assert tac(lib, h, d, LARGE) == want, k
            lib.free(h)
            if not struck:
                break
        else:
            raise AssertionError("no end")


def test_without_room_for_the_bit_sliced_form(lib):
    """The frontier form takes a batch for which the scratch or the tables of the bit-sliced form find no room; what it leaves
    is the general kernel's then.  With memory there again the next call is as on a fresh handle."""
    d = GRAPHS["wide"]()
    h = lib.build(d)[1]
    lib.tictac_trim_memory()
    before = lib.count("device_bytes")
    want = tac(lib, h, d, LARGE)
    assert want == ["tac_frontier_kernel", "tac_sliced_kernel", "tac_kernel"]
    most = lib.count("device_bytes") - before
    lib.free(h)
    taken = []
    for part in (1.0, 0.5, 0.1, 0.05, 0.02):
        h = lib.build(d)[1]
        lib.tictac_trim_memory()
        lib.host_device_limit(int(lib.count("device_bytes") + part * most))
        taken.append(tac(lib, h, d, LARGE))
        lib.host_device_limit(-1)
        assert lib.hipGetLastError() == 0
        assert tac(lib, h, d, LARGE) == want
        lib.free(h)
    assert taken[0] == want and all(t == ["tac_frontier_kernel", "tac_kernel"] for t in taken[1:]), taken


def intervals(starts, R):
    """Chains of ops with recvs a, a + 1, .. behind each other, from each of the first recvs on: the sets a .. j, one of each chain in
    the frontier at a time."""
    a, j = np.triu_indices(starts, 1, R)                # by the op before and recv j, or by recvs a and j = a + 1
    n = a.size
    col = np.stack([np.where(j == a + 1, a, R + np.arange(n) - 1), j], axis=1)
    row = np.concatenate([np.zeros(R, int), 2 * np.arange(n + 1)])
    return wl.Dag("intervals", R + n, row.astype(np.int32), col.ravel().astype(np.int32), np.arange(R, dtype=np.int32), np.ones(n), np.ones(R))


def test_capture_after_calls_that_found_no_room(lib):
    """A call under capture allocates nothing when an earlier one was at least as large, also where that one found room for one of
    the two forms only: the same kernels take it."""
    def captured(h, d, B, room):
        lib.host_forget_launches()
        lib.host_capturing(1)
        rc = lib.tac(h, d, B, room)
        lib.host_capturing(0)
        assert rc == 0 and lib.hipGetLastError() == 0, lib.error()
        return names(lib)

    def first(d, B, room, extra):
        h = lib.build(d)[1]
        lib.tictac_trim_memory()
        lib.host_device_limit(lib.count("device_bytes") + extra if extra >= 0 else -1)
        lib.host_forget_launches()
        assert lib.tac(h, d, B, room) == 0, lib.error()
        lib.host_device_limit(-1)
        return h, names(lib)

    # room for the frontier form (0.1 GB less than the other)
    d, room = GRAPHS["wide"](), {}
    h, taken = first(d, LARGE, room, 50 << 20)
    assert taken == ["tac_frontier_kernel", "tac_kernel"]
    assert captured(h, d, LARGE, room) == taken
    lib.free(h)

    # room for the bit-sliced form only: from about 86 000 classes on the other wants more, for it has more samples under way
    d, B = intervals(214, 512), 4096
    room = dict(B=B, op=np.zeros((B, d.n_compute)), rv=np.zeros((B, d.n_recv)), order=np.zeros((B, d.n_recv), np.int32),
                out=np.zeros((5, B)))                   # (never touched)
    h, taken = first(d, B, room, -1)
    assert taken == ["tac_frontier_kernel", "tac_sliced_kernel", "tac_kernel"]
    lib.free(h)
    h, taken = first(d, B, room, 700 << 20)
    assert taken == ["tac_sliced_kernel", "tac_kernel"]
    assert captured(h, d, B, room) == taken
    lib.free(h)
