"""The library's host code against a stand-in for the HIP runtime (host_lib.py): no GPU, no kernel runs."""

import ctypes
import time
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_1803_03288_amd import workloads as wl

from host_lib import HostLib, I32, build_host_lib, ptr
from test_gpu_lane_layouts import SLOTS
from test_gpu_recompute import BATCHES, lists_at
from test_gpu_tac_chain import GRAPHS as CHAINS, REFUSED, SECOND_GATES


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


# ---- memory that runs out ----

def layered(levels, width, recvs):
    return wl.layered_dag(41, levels=levels, width=width, fan_in=(1, 3), back=3, n_recv=recvs, attach=(1, 3))


def with_sends():
    """The chain of twelve jobs, and a send behind each of its compute ops."""
    d = wl.chain_dag(12)
    behind = d.compute_ids()
    k = behind.size
    row = np.concatenate([d.row_ptr, d.row_ptr[-1] + 1 + np.arange(k)]).astype(np.int32)
    col = np.concatenate([d.col_idx, behind]).astype(np.int32)
    return wl.Dag("chain_sends", d.n_ops + k, row, col, d.recv_ids, np.ones(d.n_compute + k), np.ones(d.n_recv))


GRAPHS = {
    "chain": lambda: wl.chain_dag(40),                  # rows formed on the host, TAC by chains
    "layered": lambda: layered(30, 12, 70),             # rows formed on the host, TAC in registers
    "wide": lambda: layered(16, 220, 512),              # level-major records of both kinds, bit-sliced TAC
    "device": lambda: layered(60, 220, 1280),           # rows formed on the device
}


def calls(lib, d):
    """The calls on a handle that may take memory, as ``(name, call)``."""
    B, R = 8192, d.n_recv
    room, five = {}, [np.zeros(64) for _ in range(5)]
    op, rv = np.ones((64, d.n_compute)), np.ones((64, R))
    order, chan = np.arange(R, dtype=np.int32), np.zeros(R, dtype=np.int32)
    out = [ptr(x) for x in five]
    big = d.n_ops > 2000
    yield "recompute", lambda h: lib.tictac_dag_recompute_deps(h, None)
    yield "batch", lambda h: lib.tictac_dag_recompute_deps_batch((ctypes.c_void_p * 2)(h, h), I32(2), None)
    yield "tac", lambda h: lib.tac(h, d, 300 if big else B, room)
    yield "simulate", lambda h: lib.tictac_simulate(h, I32(64), ptr(order), I32(0), ptr(op), ptr(rv), *out, None)
    if not big:
        yield "channels", lambda h: lib.tictac_simulate_channels(h, I32(64), I32(2), ptr(chan), ptr(order), I32(0), ptr(op), ptr(rv), *out, None)
    if d.name == "chain_sends":
        sends = np.arange(24, 36, dtype=np.int32)
        yield "sends", lambda h: lib.tictac_simulate_sends(h, I32(64), I32(12), ptr(sends), ptr(order), I32(0), ptr(op), ptr(rv), *out, None)


@pytest.mark.parametrize("name", list(GRAPHS) + ["sends"])
def test_no_exception_leaves_an_entry_point(lib, name):
    """Every allocation of host memory that a call makes fails once, one after the other: the call says so."""
    d = with_sends() if name == "sends" else GRAPHS[name]()

    def fails_at_each(call, done):
        for k in range(4000):
            lib.host_fail_new(k)
            rc, h = call()
            struck = lib.host_fail_new_left() < 0
            lib.host_fail_new(-1)
            if not struck:
                assert rc == 0, lib.error()
                return h
            assert rc in (0, -8), (k, rc, lib.error())          # (0: made do without)
            done(h)
        raise AssertionError("no end")

    h = fails_at_each(lambda: lib.build(d), lambda h: lib.free(h) if h.value else None)
    lib.free(h)
    for what, call in calls(lib, d):
        handles = []

        def fresh():
            lib.host_pause_failures(1)
            rc, h = lib.build(d)
            lib.host_pause_failures(0)
            assert rc == 0
            handles.append(h)
            return call(h), h
        fails_at_each(fresh, lambda h: None)
        for h in handles:
            lib.free(h)


def test_chains_planned_beside_the_class_totals(lib):
    """The tables of the chain form of a graph of more than a thousand ops and predecessors are made in two parts, the second while the
    class totals are formed: whichever allocation fails, of the device's memory or the host's, the call is taken all the same, or says so, and the
    next one is what it is on a fresh handle."""
    d = wl.chain_dag(400)
    rc, h = lib.build(d)
    lib.host_forget_launches()
    assert lib.tac(h, d, 8192) == 0
    want = [k for k in lib.kernels() if "copy_in" not in k]
    assert ["class_totals" in want[0], "tac_chain" in want[1]] == [True, True], want
    lib.free(h)
    for fail, left in ((lib.host_fail_device, lib.host_fail_device_left), (lib.host_fail_new, lib.host_fail_new_left)):
        for k in range(4000):
            rc, h = lib.build(d)
            assert lib.tictac_trim_memory() == 0
            fail(k)
            rc = lib.tac(h, d, 8192)
            struck = left() < 0
            fail(-1)
            assert rc in (0, -8) and lib.hipGetLastError() == 0, (k, rc, lib.error())
            for _ in range(2):
                lib.host_forget_launches()
                assert lib.tac(h, d, 8192) == 0, lib.error()
                assert [x for x in lib.kernels() if "copy_in" not in x] == want, (k, lib.kernels())
            lib.free(h)
            if not struck:
                break
        else:
            raise AssertionError("no end")


@pytest.mark.parametrize("name", list(REFUSED))
def test_graphs_without_the_chain_form(lib, name):
    """A graph that has more chains or gates than the chain form takes: its first call launches nothing for that form and takes no memory
    for it, whether its tables would be made at once or in two parts."""
    d = REFUSED[name]()
    B = 8192
    assert d.n_ops + d.col_idx.size > 1000
    h = lib.build(d)[1]
    lib.tictac_trim_memory()
    before = lib.count("device_bytes")
    room = {}
    for _ in range(2):
        lib.host_forget_launches()
        assert lib.tac(h, d, B, room) == 0, lib.error()
        first, *rest = lib.kernels()
        assert "tac_reg_kernel" in first and len(rest) == 1 and "10tac_kernel" in rest[0], lib.kernels()
        assert 4 * B <= lib.count("device_bytes") - before <= 5 * B         # (a flag per sample, an eighth more)
    lib.free(h)


@pytest.mark.parametrize("name", list(GRAPHS) + ["sends"])
def test_a_failed_allocation_leaves_nothing_behind(lib, name):
    """Every allocation of device memory that a call makes fails once, one after the other, and so does every one of host
    memory: the next call on the handle launches what it launches on a fresh one, and a freed handle's blocks serve the
    next handle."""
    d = with_sends() if name == "sends" else GRAPHS[name]()
    fail = {"device": (lib.host_fail_device, lib.host_fail_device_left), "new": (lib.host_fail_new, lib.host_fail_new_left)}

    def kernels(call, h):
        lib.host_forget_launches()
        assert call(h) == 0, lib.error()
        tables = ("copy_in", "sliced_colbits", "sliced_planes")         # (made once per handle)
        return [k for k in lib.launches() if not any(t in k[0] for t in tables)]

    for what, call in calls(lib, d):
        rc, h = lib.build(d)
        want = kernels(call, h)
        lib.free(h)
        for kind, (order, left) in fail.items():
            for k in range(4000):
                rc, h = lib.build(d)
                assert rc == 0
                assert lib.tictac_trim_memory() == 0            # (so that the call allocates)
                order(k)
                rc = call(h)
                struck = left() < 0
                order(-1)
                assert rc in (0, -7, -8), (what, kind, k, lib.error())
                assert lib.hipGetLastError() == 0, (what, kind, k)
                assert kernels(call, h) == want, (what, kind, k)
                lib.free(h)
                if not struck:
                    break
    rc, h = lib.build(d)
    lib.free(h)
    allocs = lib.count("allocs")
    rc, h = lib.build(d)
    lib.free(h)
    assert lib.count("allocs") == allocs
    lib.tictac_trim_memory()
    assert lib.count("device_bytes") == 0


def test_tac_makes_do_with_the_memory_there_is(lib):
    """The chain form takes a call in smaller chunks when the device has no room for a large one, and leaves it to the
    register-resident kernel when it has none for 8 192 samples or for the tables."""
    d = wl.chain_dag(40)
    B = 1 << 16
    room = {}

    def run(limit, h=None):
        rc, fresh = (0, h) if h is not None else lib.build(d)
        lib.tictac_trim_memory()
        lib.host_forget_launches()
        lib.host_device_limit(limit if limit < 0 else lib.count("device_bytes") + limit)
        rc = lib.tac(fresh, d, B, room)
        lib.host_device_limit(-1)
        assert rc == 0, lib.error()
        assert lib.hipGetLastError() == 0
        return fresh, lib.kernels()

    h, all_of_it = run(-1)
    assert sum("class_totals" in k for k in all_of_it) == 1
    lib.free(h)
    flags = 4 * B
    for limit, chunks in ((40 << 20, 2), (14 << 20, 4), (flags + (7 << 20), 8), (flags + (5 << 20), 0), (flags * 2, 0)):
        h, kernels = run(limit)
        assert sum("class_totals" in k for k in kernels) == chunks, (limit, kernels)
        assert sum("tac_reg_kernel" in k for k in kernels) == (chunks == 0), (limit, kernels)
        assert run(-1, h)[1][-3:] == all_of_it[-3:]           # with memory there again: as on a fresh handle
        lib.free(h)


def test_a_workspace_leaves_room_for_the_tables(lib):
    """Whatever memory there is, the class totals are formed only where the chains come after them."""
    d, B, room = wl.chain_dag(400), 16384, {}

    def run(limit):
        h = lib.build(d)[1]
        lib.tictac_trim_memory()
        before = lib.count("device_bytes")
        lib.host_device_limit(before + limit if limit >= 0 else -1)
        lib.host_forget_launches()
        assert lib.tac(h, d, B, room) == 0, lib.error()
        lib.host_device_limit(-1)
        taken, kernels = lib.count("device_bytes") - before, lib.kernels()
        lib.free(h)
        return taken, tuple(sum(k in x for x in kernels) for k in ("class_totals", "tac_chain", "tac_reg"))
    most, launches = run(-1)
    assert launches == (1, 1, 0)
    for some in (most, most // 2):                  # (of one chunk and of two)
        for kib in range(0, 240, 4):
            launches = run(some - (kib << 10))[1]
            assert launches in ((1, 1, 0), (2, 2, 0), (0, 0, 1)), (some, kib, launches)


@pytest.mark.parametrize("name", list(GRAPHS))
def test_the_first_propagation_finds_its_tables_made(lib, name):
    """recompute_deps on a handle that has just been built allocates nothing, waits for nothing and can be captured; the
    same for several handles waits for nothing."""
    d = GRAPHS[name]()
    rc, h = lib.build(d)
    rc, other = lib.build(d)
    before = {what: lib.count(what) for what in ("waits", "allocs", "new")}
    lib.host_capturing(1)
    rc = lib.tictac_dag_recompute_deps(h, None)
    lib.host_capturing(0)
    assert rc == 0, lib.error()
    assert before == {what: lib.count(what) for what in before}
    assert lib.tictac_dag_recompute_deps_batch((ctypes.c_void_p * 2)(h, other), I32(2), None) == 0
    assert before["waits"] == lib.count("waits")
    lib.free(h)
    lib.free(other)


@pytest.mark.parametrize("recvs,at,kernel", [(60, 256, "propagate_levelsILi1E"), (60, 257, "wideILi1E"), (60, 1024, "wideILi1E"),
                                             (128, 288, "propagate_nodesILi2E"), (128, 289, "wideILi2E"), (200, 256, "propagate_nodesILi4E"),
                                             (1024, 256, "propagate_levelsILi1E"), (1024, 257, "wideILi1E"), (2000, 800, "wideILi1E"),
                                             (2000, 1025, "wideILi1E")])
def test_graphs_with_wide_levels_are_propagated(lib, recvs, at, kernel):
    """Levels that one pass of a workgroup takes, but not the records of the chunked kernel: the kernel for wider levels."""
    d = wl.layered_dag(3, levels=24, width=at, fan_in=(2, 3), back=1, n_recv=recvs, attach=(1, 2))
    rc, h = lib.build(d)
    assert rc == 0, lib.error()
    lib.host_forget_launches()
    assert lib.tictac_dag_recompute_deps(h, None) == 0, lib.error()
    (name, _, _, lds, _), = [l for l in lib.launches() if "propagate" in l[0]]
    assert kernel in name and lds <= 150 * 1024, (name, lds)
    lib.free(h)


@pytest.mark.parametrize("name", ["chain", "wide", "device"])
def test_a_first_tac_call_waits_for_nothing_of_the_callers(lib, name):
    """The tables that a first TAC call makes go to the device without a wait for the caller's stream or the device."""
    d = GRAPHS[name]()
    rc, h = lib.build(d)
    waits = lib.count("waits")
    assert lib.tac(h, d, 8192 if name == "chain" else 300) == 0
    assert lib.count("waits") == waits
    lib.free(h)


def test_a_first_tac_call_under_capture(lib):
    """Chain tables cannot be made on a stream that is being captured: the register-resident kernel takes the call, as far
    as the workspace reaches, and the next call outside makes them."""
    d = GRAPHS["chain"]()
    rc, h = lib.build(d)
    assert lib.tac(h, d, 8190) == 0                 # (one sample short of the chain form, two of its workspace)
    lib.host_forget_launches()
    lib.host_capturing(1)
    rc = lib.tac(h, d, 8192)
    lib.host_capturing(0)
    assert rc == 0, lib.error()
    assert any("tac_reg" in k for k in lib.kernels()) and not any("chain" in k for k in lib.kernels())
    lib.host_forget_launches()
    assert lib.tac(h, d, 8192) == 0 and any("tac_chain" in k for k in lib.kernels())
    lib.host_forget_launches()
    lib.host_capturing(1)
    assert lib.tac(h, d, 8192) == 0 and any("tac_chain" in k for k in lib.kernels())
    lib.host_forget_launches()
    assert lib.tac(h, d, 8256) == 0 and any("tac_reg" in k or "tac_chain" in k for k in lib.kernels())
    lib.host_capturing(0)
    lib.free(h)


@pytest.mark.parametrize("name,B,waves", [("k13", 1, 8), ("k13", 2048, 8), ("k13", 2049, 16), ("k15", 3000, 8), ("k15", 4000, 8),
                                          ("k15", 4097, 16), ("wide", 9000, 8), ("k6", 1, 16)])
def test_waves_of_tac_in_registers(lib, name, B, waves):
    """More than eight classes per lane: the kernel of eight waves with all registers where it takes no more sets than as many waves
    as LDS holds: at least twelve with k13, ten with k15, fewer than eight with wide."""
    d = wl.layered_dag(17, levels=44, width=20, fan_in=(1, 4), back=3, n_recv=640, attach=(1, 8)) if name == "wide" else SLOTS[name]()
    h = lib.build(d)[1]
    classes = I32()
    lib.tictac_dag_info(h, None, None, None, None, ctypes.byref(classes))
    assert (classes.value > 512) == (name != "k6") and classes.value <= 1024, classes.value
    lib.host_forget_launches()
    assert lib.tac(h, d, B) == 0, lib.error()
    (name, _, threads, lds, _), = [l for l in lib.launches() if "tac_reg" in l[0]]
    assert f"ELi{waves}E" in name and threads <= 64 * waves and lds <= 150 * 1024, (name, threads, lds)
    lib.free(h)


@pytest.mark.parametrize("each", [1, 3, 4, 5, 6, 8, 9, 13])
@pytest.mark.parametrize("slots,dag", [(1, lambda: layered(12, 5, 20)), (3, wl.resnet50_dag), (4, lambda: layered(20, 14, 200))])
def test_full_workgroups_of_tac_in_registers(lib, slots, dag, each):
    """Up to four classes per lane several workgroups of four waves share a compute unit: no more of them than take the samples."""
    d = dag()
    h = lib.build(d)[1]
    B = 256 * each - 3
    lib.host_forget_launches()
    assert lib.tac(h, d, B) == 0, lib.error()
    (name, blocks, threads, _, _), = [l for l in lib.launches() if "tac_reg" in l[0]]
    assert f"tac_reg_kernelILi{slots}E" in name and threads == 256
    assert blocks == min(256 * 4, -(-B // min(4, each))), (name, blocks)
    lib.free(h)


def test_many_recvs_without_room_for_flags(lib):
    """A graph with more than 384 recvs, whose general kernel needs no workspace, is taken without one: on a stream that is
    being captured, and where the device has no memory left."""
    d = wl.layered_dag(17, levels=8, width=8, fan_in=(1, 3), back=3, n_recv=400, attach=(1, 4))
    rc, h = lib.build(d)

    def which():
        lib.host_forget_launches()
        rc = lib.tac(h, d, 50)
        assert rc == 0, lib.error()
        return ["tac_reg" if "tac_reg" in k else "tac" for k in lib.kernels() if "tac" in k]

    lib.host_capturing(1)
    assert which() == ["tac"]
    lib.host_capturing(0)
    lib.tictac_trim_memory()
    lib.host_device_limit(lib.count("device_bytes"))
    assert which() == ["tac"]
    lib.host_device_limit(-1)
    assert which() == ["tac_reg", "tac"]
    lib.host_capturing(1)
    assert which() == ["tac_reg", "tac"]
    lib.host_capturing(0)
    lib.free(h)


@pytest.mark.parametrize("name", list(CHAINS))
def test_chain_form_and_second_gates(lib, name):
    """Every graph of the chain form's tests takes it, those with recvs that are sinks of two gates the kernels that know of them."""
    d = CHAINS[name]()
    h = lib.build(d)[1]
    lib.host_forget_launches()
    assert lib.tac(h, d, 8192) == 0, lib.error()
    kernel, = [k for k in lib.kernels() if "tac_chain_kernel" in k]
    slots, second = int(kernel[kernel.index("ILi") + 3]), "ELb1E" in kernel
    assert second == (name in SECOND_GATES) and slots == SECOND_GATES.get(name, slots), kernel
    lib.free(h)


def out_of_order(degrees, seed=2):
    """An op per entry of ``degrees`` behind four recvs, with so many predecessors among the ops before it."""
    g = np.random.default_rng(seed)
    row, col = [0] * 5, []
    for k, n in enumerate(degrees):
        col += sorted(g.choice(4 + k, size=min(n, 4 + k), replace=False).tolist())
        row.append(len(col))
    n = 4 + len(degrees)
    return wl.Dag("degrees", n, np.array(row, np.int32), np.array(col, np.int32), np.arange(4, dtype=np.int32), np.ones(len(degrees)), np.ones(4))


# numbers of predecessors that vary from op to op, and that do not; a few ops and many
@pytest.mark.parametrize("count", [3, 795, 796, 5000])
@pytest.mark.parametrize("degrees", [(1, 4, 2, 3), (2,), (3, 3, 3, 1), (1, 2, 9, 3), (0, 4, 3, 5)])
def test_predecessors_are_checked(lib, count, degrees):
    """A predecessor out of range is refused with its place, whichever of an op's it is; one with the op's own or a higher id is not,
    unless that makes a cycle."""
    d = out_of_order([degrees[k % len(degrees)] for k in range(count)])
    rc, h = lib.build(d)
    assert rc == 0, lib.error()
    lib.free(h)
    g = np.random.default_rng(count)
    for v in g.choice(np.arange(4, d.n_ops), size=min(count, 6), replace=False):
        for e in range(d.row_ptr[v], d.row_ptr[v + 1]):
            for bad in (-1, d.n_ops, -2**31, 2**31 - 1):
                col = d.col_idx.copy()
                col[e] = bad
                rc, _ = lib.build(wl.Dag("bad", d.n_ops, d.row_ptr, col, d.recv_ids, d.op_median, d.recv_bytes))
                assert rc == -2 and lib.error() == f"pred_col_idx[{e}]={bad} out of range"
            col = d.col_idx.copy()
            col[e] = v
            assert lib.build(wl.Dag("self", d.n_ops, d.row_ptr, col, d.recv_ids, d.op_median, d.recv_bytes))[0] == -3
    # the other way round: every predecessor has a higher id
    n = d.n_ops
    rows = [(n - 1 - d.col_idx[d.row_ptr[v]:d.row_ptr[v + 1]])[::-1] for v in range(n)][::-1]
    back = wl.Dag("back", n, np.cumsum([0] + [len(r) for r in rows]).astype(np.int32), np.concatenate(rows).astype(np.int32),
                  (n - 1 - d.recv_ids)[::-1].astype(np.int32).copy(), d.op_median, d.recv_bytes)
    levels = []
    for x in (d, back):
        rc, h = lib.build(x)
        assert rc == 0, lib.error()
        got = I32()
        lib.tictac_dag_info(h, None, None, None, ctypes.byref(got), None)
        levels.append(got.value)
        lib.free(h)
    assert levels[0] == levels[1]


def three_inputs(levels, width, far, wide, recvs, idle):
    """Three inputs per op from the two levels before; every ``far``-th op one from the first level as well, every ``wide``-th six;
    ``idle`` further recvs without a use."""
    row, col = [0] * (recvs + idle + 1), []
    for v in range(levels * width):
        l, w = divmod(v, width)
        ins = {v % recvs} if l == 0 else {recvs + idle + max(0, l - 1 - k % 2) * width + (w + 7 * k) % width for k in range(6 if v % wide == 0 else 3)}
        if l and v % far == 0:
            ins.add(recvs + idle + w)
        col += sorted(ins)
        row.append(len(col))
    n = recvs + idle + levels * width
    return wl.Dag("three_inputs", n, np.array(row, np.int32), np.array(col, np.int32), np.arange(recvs + idle, dtype=np.int32),
                  np.ones(levels * width), np.ones(recvs + idle))


@pytest.mark.parametrize("far,wide,fits", [(1 << 30, 1 << 30, True), (1000, 1 << 30, True), (1 << 30, 500, True), (100, 300, True), (10, 20, False)])
def test_room_for_the_lists_of_the_level_kernel(lib, far, wide, fits):
    """Nodes that fit no record (more inputs than it has room for, or one that has left the ring) have lists; LDS has room for all of
    them, or for none where they are too many, whether the host makes the records or a kernel does."""
    most = {}
    for idle in (0, 192):
        d = three_inputs(280, 100, far, wide, 1080, idle)
        on_host = (d.n_ops + d.n_edges) * ((d.n_recv + 63) // 64) <= 1 << 21
        handles = [lib.build(d) for _ in range(3)]
        assert [rc for rc, _ in handles] == [0, 0, 0], lib.error()
        arr = (ctypes.c_void_p * 3)(*[h for _, h in handles])
        lib.host_forget_launches()
        assert lib.tictac_dag_recompute_deps_batch(arr, I32(3), None) == 0, lib.error()
        most[on_host], = [lds for name, _, _, lds, _ in lib.launches() if "propagate_levels_batch" in name]
        for _, h in handles:
            lib.free(h)
    ring = most[True] // 8192 * 8192 + 16       # (of one-word slices: 1 024 slots and more, two words of zeros)
    lists = (most[True] - ring) // 4
    assert most[True] == most[False] and lists == (0 if far == wide or not fits else lists) <= 4096
    assert (lists > 0) == (fits and far != wide)


@pytest.mark.parametrize("recvs,run,slots,quads", [(250, 80, 4, False), (290, 16, 5, False), (290, 40, 5, False), (290, 64, 5, True),
                                                   (380, 16, 6, False), (380, 64, 6, True), (440, 2, 7, False), (440, 64, 7, True),
                                                   (500, 1, 8, False), (500, 90, 8, True)])
def test_class_totals_by_quads_where_columns_have_long_runs(lib, recvs, run, slots, quads):
    """Four lanes are compared only where many columns next to each other have one class and, in the simulation by waves, where several
    workgroups share a compute unit: elsewhere that costs more than it gives."""
    b = wl._Builder()
    for r in [b.recv(1e5) for _ in range(recvs)]:
        for _ in range(run):
            r = b.op([r], 1e-4, "op")
    d = b.finish("runs", seed=3, batch=4)
    rc, h = lib.build(d)
    assert rc == 0, lib.error()
    chan = np.zeros(recvs, np.int32)
    room = np.zeros(1)                      # (no kernel runs: what the samples are is no matter)
    for B in (8, 1024, 1025):
        lib.host_forget_launches()
        out = [ptr(room)] * 5
        assert lib.tictac_simulate(h, I32(B), ptr(room), I32(recvs), ptr(room), ptr(room), *out, None) == 0, lib.error()
        assert lib.tictac_simulate_channels(h, I32(B), I32(2), ptr(chan), ptr(room), I32(recvs), ptr(room), ptr(room), *out, None) == 0
        one, several = [k for k in lib.kernels() if "simulate_" in k]
        assert f"simulate_wave_kernelILi{slots}ELi{3 if quads and B > 1024 else 1}E" in one
        assert f"simulate_channels_kernelILi{slots}ELNS_4SumsE{1 if quads else 0}E" in several
    lib.free(h)


@pytest.mark.parametrize("width,recvs,B,kernel", [(130, 100, 1, "simulate_kernelILi1024E"), (130, 100, 256, "simulate_kernelILi1024E"),
                                                  (130, 100, 257, "simulate_wave"), (50, 100, 1, "simulate_wave"),
                                                  (220, 64, 1, "simulate_wave")])
def test_small_batches_with_an_order_each(lib, width, recvs, B, kernel):
    """Graphs of more than 2 048 classes and rows of two words or more, no more samples than compute units: a workgroup per sample."""
    d = layered(40, width, recvs)
    h = lib.build(d)[1]
    classes = I32()
    lib.tictac_dag_info(h, None, None, None, None, ctypes.byref(classes))
    assert (classes.value > 2048) == (width > 50)
    op, rv, order = np.ones((B, d.n_compute)), np.ones((B, recvs)), np.tile(np.arange(recvs, dtype=np.int32), (B, 1))
    out = [np.zeros(B) for _ in range(5)]
    lib.host_forget_launches()
    assert lib.tictac_simulate(h, I32(B), ptr(order), I32(recvs), ptr(op), ptr(rv), *(ptr(x) for x in out), None) == 0, lib.error()
    assert any(kernel in k for k in lib.kernels()), lib.kernels()
    lib.free(h)


def test_one_order_without_room_for_a_word_per_column(lib):
    """One order for all samples on a stream that is being captured: a workspace that holds a word per class but not per
    column serves the call, by class."""
    d = wl.layered_dag(17, levels=40, width=30, fan_in=(1, 3), back=3, n_recv=100, attach=(1, 4))
    rc, h = lib.build(d)
    B = 256
    op, rv, order = np.ones((B, d.n_compute)), np.ones((B, d.n_recv)), np.arange(d.n_recv, dtype=np.int32)
    out = [np.zeros(B) for _ in range(5)]

    def which():
        lib.host_forget_launches()
        rc = lib.tictac_simulate(h, I32(B), ptr(order), I32(0), ptr(op), ptr(rv), *(ptr(x) for x in out), None)
        assert rc == 0, lib.error()
        return [name for name in ("simulate_wave", "simulate_kernel") if any(name in k for k in lib.kernels())]

    assert lib.tac(h, d, 1000) == 0             # (leaves a word per sample)
    lib.host_capturing(1)
    assert which() == ["simulate_kernel"]
    lib.host_capturing(0)
    assert which() == ["simulate_wave"]
    lib.host_capturing(1)
    assert which() == ["simulate_wave"]
    lib.host_capturing(0)
    lib.free(h)


def test_handles_do_not_wait_for_each_others_tables(lib):
    """Four threads make the tables of a handle each while every copy takes 0.2 s: side by side, not one after the other."""
    d = GRAPHS["chain"]()
    handles = [lib.build(d)[1] for _ in range(4)]
    rooms = [{} for _ in range(4)]

    with ThreadPoolExecutor(4) as ex:
        assert list(ex.map(lambda k: lib.tac(handles[k], d, 8190, rooms[k]), range(4))) == [0] * 4
        lib.host_forget_launches()
        lib.host_slow_copies(200000)
        start = time.perf_counter()
        assert list(ex.map(lambda k: lib.tac(handles[k], d, 8192, rooms[k]), range(4))) == [0] * 4
        took = time.perf_counter() - start
    lib.host_slow_copies(0)
    assert sum("copy_in" in k for k in lib.kernels()) == 4
    assert took < 0.6
    for h in handles:
        lib.free(h)


def test_kept_memory_is_bounded_and_given_back(lib):
    """Threads that come and go leave no pinned memory of their own behind, and everything kept from freed handles can be
    given back while another handle lives on."""
    lib.tictac_trim_memory()
    assert lib.count("device_bytes") == lib.count("pinned_bytes") == 0
    d = GRAPHS["wide"]()
    for _ in range(6):
        with ThreadPoolExecutor(1) as ex:
            lib.free(ex.submit(lib.build, d).result()[1])
    assert 0 < lib.count("pinned_bytes") <= 4 << 20
    rc, h = lib.build(d)
    lib.free(lib.build(d)[1])
    held = lib.count("device_bytes")
    assert lib.tictac_trim_memory() == 0
    assert 0 < lib.count("device_bytes") < held and lib.count("pinned_bytes") == 0
    assert lib.tac(h, d, 300) == 0
    lib.free(h)
    assert lib.tictac_trim_memory() == 0 and lib.count("device_bytes") == 0
    # no more than the bound is kept
    handles = []
    for _ in range(16):
        handles.append(lib.build(d)[1])
        assert lib.tac(handles[-1], d, 512) == 0
    assert lib.count("device_bytes") > 2 << 30
    for h in handles:
        lib.free(h)
    assert 1 << 29 < lib.count("device_bytes") <= 1 << 30
    lib.tictac_trim_memory()


@pytest.mark.parametrize("C,R,B,words", [
    (1025, 600, 4096, 1), (28672, 2048, 4096, 1), (28673, 2048, 4096, 2), (30119, 4096, 4096, 2), (44588, 2048, 4096, 2),
    (57344, 4096, 4096, 2), (57345, 4096, 4096, 3), (62837, 4096, 4096, 3), (86016, 4096, 4096, 3),
    (86017, 4096, 4096, 2),                                     # too many for two workgroups of three words: the fewest
    (122881, 4096, 4096, 3), (30119, 4096, 256, 1), (53188, 4096, 256, 1), (62837, 4096, 256, 2), (62837, 4096, 257, 3)])
def test_two_workgroups_of_the_sliced_kernel_share_a_compute_unit_where_they_fit(lib, C, R, B, words):
    """Words per lane: the fewest with which two workgroups fit a compute unit, on small graphs as on the largest; the
    fewest at all where there are no two samples per compute unit or no such number up to three."""
    lib.tictac_trim_memory()
    lib.host_forget_launches()
    assert lib.host_tac_sliced(C, R, B) == 0
    (name, blocks, threads, lds, _), = lib.launches()
    assert f"tac_sliced_kernelILi{words}E" in name, name
    assert (threads // 64 - 1) * 64 * 64 * words >= C
    assert blocks == min(B, 256 * min(160 * 1024 // lds, 16 // (threads // 64)))


# nine inputs at one node in so many: of the level before (none leaves the ring), of 18 levels before (77 and 163 from beyond a ring of
# sixteen levels, at 8 000 nodes: the nodes that follow such a node are at higher levels themselves)
@pytest.mark.parametrize("every,back,stored", [(1 << 30, 1, True), (9, 1, True), (60, 18, True), (30, 18, False)])
def test_batches_of_graphs_with_far_inputs(lib, every, back, stored):
    """The computing waves store the rows of graphs whose lists name more than one row from memory per hundred nodes."""
    d = lists_at(80, 100, every, back)
    h = lib.build(d)[1]
    lib.host_forget_launches()
    assert lib.tictac_dag_recompute_deps_batch((ctypes.c_void_p * 3)(h, h, h), I32(3), None) == 0, lib.error()
    kernel = [k for k in lib.kernels() if "propagate" in k][0]
    assert ("propagate_levels_q_stored" if stored else "propagate_levels_q_batch") in kernel, kernel
    lib.free(h)


# two workgroups per graph;  1 000 list entries, which LDS holds, and 6 000
@pytest.mark.parametrize("every", [120, 20])
def test_batches_of_graphs_with_many_list_entries(lib, every):
    """Lists that LDS does not hold: the computing waves store the rows of 8 to 56 workgroups if their number is a multiple of eight, and of 32 to 63."""
    h = lib.build(lists_at(120, 100, every, 1))[1]
    for n in (4, 5, 8, 15, 16, 17, 20, 28, 31, 32):
        lib.host_forget_launches()
        assert lib.tictac_dag_recompute_deps_batch((ctypes.c_void_p * n)(*[h] * n), I32(n), None) == 0, lib.error()
        (kernel, blocks, *_), = [l for l in lib.launches() if "propagate" in l[0]]
        assert blocks == 2 * n
        assert ("propagate_levels_q_stored" in kernel) == (every == 120 or n in (5, 15, 32)), (n, kernel)
    lib.free(h)


# four workgroups per graph.  60 x 200 ops: 256 MiB are 74 graphs, 600 MiB 174;  600 x 50: 1.5 TB/s are 68 graphs, 600 MiB 76
@pytest.mark.parametrize("levels,width,every,through", [(60, 200, 1 << 30, (76, 78, 174)), (60, 200, 9, ()), (600, 50, 1 << 30, (72, 74, 76))])
def test_batches_whose_rows_go_through_the_caches(lib, levels, width, every, through):
    """Rows beyond what the Infinity Cache holds are stored through the caches where many workgroups, a multiple of eight, form them fast; past the
    caches where lists come from memory."""
    d = lists_at(levels, width, every, 1, 2048)
    h = lib.build(d)[1]
    most = (600 << 20) // (d.n_ops * 32 * 8)
    for n in (30, 64, 72, 73, 74, 75, 76, 77, 78, 79, 174, 175):
        lib.host_forget_launches()
        assert lib.tictac_dag_recompute_deps_batch((ctypes.c_void_p * n)(*[h] * n), I32(n), None) == 0, lib.error()
        kernel = [k for k in lib.kernels() if "propagate" in k][0]
        want = "stored<4, false>" if n in through else "stored<4, true>" if n <= most else "batch<4>"
        got = kernel.replace("ILi4ELb1E", "<4, true>").replace("ILi4ELb0E", "<4, false>").replace("ILi4E", "<4>")
        assert "propagate_levels_q_" + want in got, (n, kernel)
    lib.free(h)


@pytest.mark.parametrize("name", list(BATCHES))
def test_which_kernel_takes_several_graphs(lib, name):
    """Two waves more store the rows of graphs with up to 224 slots per level, up to 600 MiB of rows; beyond, and of graphs with wider
    levels or lists of rows that have left the ring, those that compute."""
    d, most = BATCHES[name]()
    h = lib.build(d)[1]
    each = d.n_ops * ((d.n_recv + 63) // 64) * 8
    limit = (600 << 20) // each
    slots = {}
    for n in (2, limit, limit + 1):
        lib.host_forget_launches()
        assert lib.tictac_dag_recompute_deps_batch((ctypes.c_void_p * n)(*[h] * n), I32(n), None) == 0, lib.error()
        (kernel, blocks, threads, lds, _), = [l for l in lib.launches() if "propagate" in l[0]]
        stored = "25propagate_levels_q_storedILi4E" in kernel
        assert stored or "24propagate_levels_q_batchILi4E" in kernel, kernel
        assert stored == (most and n <= limit), (n, kernel)
        compute = threads - (128 if stored else 0)
        assert compute % 128 == 0 and compute <= (896 if stored else 1024) and lds <= 150 * 1024
        assert blocks == n * ((d.n_recv + 63) // 64) // 8
        slots.setdefault(stored, set()).add((compute, lds - (2 * compute if stored else 0)))
    assert len(set.union(*slots.values())) == 1, slots          # the same ring and lists; two halves of a word per slot beside them
    lib.free(h)
