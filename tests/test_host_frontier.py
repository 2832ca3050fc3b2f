"""Host side of the frontier form of TAC, against the stand-in for the HIP runtime: which calls take it, memory that runs out
while its tables are made, and streams under capture."""

import ctypes

import numpy as np
import pytest

from paper_1803_03288_amd import workloads as wl

from host_lib import I32, ptr
from test_gpu_tac_frontier import GRAPHS as LISTS, backwards
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


def in_order(d):
    """The ops, each after those before it."""
    if all((d.col_idx[d.row_ptr[v]:d.row_ptr[v + 1]] < v).all() for v in range(d.n_ops)):
        return range(d.n_ops)
    done, out = np.zeros(d.n_ops, bool), []
    for v in range(d.n_ops):
        todo = [v]
        while todo:
            u = todo[-1]
            before = [] if done[u] else [w for w in d.col_idx[d.row_ptr[u]:d.row_ptr[u + 1]] if not done[w]]
            todo += before
            if not before:
                todo.pop()
                out += [] if done[u] else [u]
                done[u] = True
    return out


def plan_of(lib, d, pieces):
    """The plan of graph ``d`` with the sets of its compute ops as classes, each in ``pieces`` of consecutive ops, and what it was made
    from: ``(plan or None, dep of the classes, class of every op, columns by class)``."""
    n, R = d.n_ops, d.n_recv
    recv_of, cls_of, level, deps = np.full(n, -1, np.int32), np.full(n, -1, np.int32), np.zeros(n, np.int32), [0] * n
    recv_of[d.recv_ids] = np.arange(R)
    members = {}
    for v in in_order(d):
        before = d.col_idx[d.row_ptr[v]:d.row_ptr[v + 1]]
        level[v] = 1 + max((level[u] for u in before), default=-1)
        for u in before:
            deps[v] |= deps[u]
        if recv_of[v] >= 0:
            deps[v] |= 1 << int(recv_of[v])
        else:
            members.setdefault(deps[v], []).append(v)
    dep, columns = [], []
    column = np.cumsum(recv_of < 0) - 1
    for bits, ops in sorted(members.items(), key=lambda m: min(m[1])):
        for part in np.array_split(np.sort(ops), min(pieces, len(ops))):
            cls_of[part] = len(dep)
            dep.append(bits)
            columns.append(column[part].tolist())
    col_cls, cnt0 = cls_of[recv_of < 0], [b.bit_count() for b in dep]
    arrays = [np.ascontiguousarray(x, np.int32) for x in (d.row_ptr, d.col_idx, level, cls_of, recv_of, cnt0, col_cls)]
    lib.L.host_frontier_plan.restype = ctypes.c_void_p
    lib.L.host_frontier_array.restype = ctypes.c_int64
    plan = lib.L.host_frontier_plan(I32(n), I32(R), I32(len(dep)), I32(col_cls.size), *(ptr(a) for a in arrays))
    if not plan:
        return None, dep, cls_of, columns
    got = {}
    for name in ("row", "inputs", "outputs", "counters", "wide", "roots", "free_cols", "own_ptr", "own", "cls_of"):
        at = ctypes.c_void_p()
        k = lib.L.host_frontier_array(ctypes.c_void_p(plan), name.encode(), ctypes.byref(at))
        got[name] = np.ctypeslib.as_array(ctypes.cast(at, ctypes.POINTER(ctypes.c_int32)), (k,)).copy() if k else np.zeros(0, np.int32)
    lib.L.host_frontier_table.restype = ctypes.c_void_p
    lib.L.host_frontier_table_array.restype = ctypes.c_int64
    table = ctypes.c_void_p(lib.L.host_frontier_table(ctypes.c_void_p(plan)))
    for i, name in enumerate(("table", "table_inputs")):
        at = ctypes.c_void_p()
        k = lib.L.host_frontier_table_array(table, I32(i), ctypes.byref(at))
        got[name] = np.ctypeslib.as_array(ctypes.cast(at, ctypes.POINTER(ctypes.c_int32)), (k,)).copy() if k else np.zeros(0, np.int32)
    lib.L.host_frontier_table_free(table)
    lib.L.host_frontier_free(ctypes.c_void_p(plan))
    return got, dep, cls_of, columns


FILL, WIDE, ONLY, LAST = 1 << 18, 1 << 19, 1 << 30, 1 << 31


@pytest.mark.parametrize("name,pieces", [("layered", 1), ("layered", 3), ("in4", 1), ("in5", 1), ("in15", 1), ("in16", 1), ("in61", 1),
                                         ("in64", 2), ("q127", 1), ("frontier300", 1), ("long_classes", 2)])
def test_the_plan_of_the_class_graph(lib, name, pieces):
    """dep of a class is the union of its inputs', none of which another one holds; outputs, counters, the classes of every recv, roots
    and columns say the same."""
    d = layered(12, 160, 300) if name == "layered" else LISTS[name]()
    p, dep, _, columns = plan_of(lib, d, pieces)
    assert p is not None
    R, C, row = d.n_recv, len(dep), p["row"].reshape(-1, 16)
    assert row.shape[0] == C
    inputs, outputs, own = [], [set() for _ in range(C)], [[] for _ in range(R)]
    for c in range(C):
        more = int(row[c, 8])
        x = np.array(inputs_of(row, p, R, c), dtype=np.int64)
        assert x.size <= 64 and (np.diff(x) > 0).all() and (more & 15) == max(0, -(-x.size // 4) - 1)
        sets = [dep[v] if v >= 0 else 1 << int(~v) for v in x]
        union = 0
        for b in sets:
            union |= b
        assert union == dep[c], c
        inputs.append(x.tolist())
        for v in x:
            if v >= 0:
                outputs[v].add(c)
            else:
                own[~v].append(c)
        for v in x[x >= 0]:                 # (no input of an input)
            assert not set(inputs_of(row, p, R, v)) & set(x.tolist()), (c, v)
    assert p["own_ptr"].tolist() == np.cumsum([0] + [len(o) for o in own]).tolist()
    assert p["own"].tolist() == [c for o in own for c in o]
    open_ = [sum(v >= 0 for v in x) for x in inputs]
    words, wide = p["counters"].astype(np.int64) & 0xffffffff, p["wide"].tolist()
    assert wide == [c for c in range(C) if open_[c] > 15] and words.size % 4 == 0
    for c in range(C):
        assert (words[c >> 3] >> (c & 7) * 4) & 15 == (open_[c] if open_[c] < 16 else 0)
    assert words[(C + 7) // 8:(C + 7) // 8 + len(wide)].tolist() == [open_[c] for c in wide]
    assert p["roots"].tolist() == [c for c in range(C) if dep[c] and not open_[c]]
    assert p["free_cols"].tolist() == [j for c in range(C) if not dep[c] for j in columns[c]]
    order = [j for c in range(C) for j in columns[c]]
    for c in range(C):
        fours, at = [row[c, 4:8].view(np.uint32).tolist()], int(row[c, 9])
        while not fours[-1][0] & LAST:
            fours.append(p["outputs"][at:at + 4].view(np.uint32).tolist())
            at += 4
        assert len({bool(z & LAST) for z in fours[-1]}) == 1 and not any(z & LAST for f in fours[:-1] for z in f)
        got = []
        for z in (z for f in fours for z in f):
            if z & FILL:
                continue
            o = wide[z & 0x3ffff] if z & WIDE else z & 0x3ffff
            assert bool(z & ONLY) == (open_[o] == 1) and bool(z & WIDE) == (open_[o] > 15)
            got.append(o)
        assert len(got) == len(set(got)) and set(got) == outputs[c], c
        n, first = int(row[c, 12]), int(row[c, 13])
        assert order[first:first + n] == columns[c] and row[c, 14:16].tolist() == (columns[c] + [0, 0])[:2]


def far_apart():
    """Fifty thousand classes between a class and two that have it among their inputs: more than the kernel's row can say."""
    d = wl.layered_dag(5, levels=500, width=160, fan_in=(1, 4), back=3, n_recv=2500, attach=(1, 8))
    recv = np.zeros(d.n_ops, bool)
    recv[d.recv_ids] = True
    head = next(v for v in range(d.n_ops) if not recv[v] and d.row_ptr[v + 1] > d.row_ptr[v])
    last = d.n_ops - 1
    more = [[head, last], [head, last, int(d.recv_ids[-1])]]
    return wl.Dag("far_apart", d.n_ops + 2, np.concatenate([d.row_ptr, d.row_ptr[-1] + np.cumsum([len(m) for m in more])]).astype(np.int32),
                  np.concatenate([d.col_idx, *more]).astype(np.int32), d.recv_ids, np.ones(d.n_compute + 2), d.recv_bytes)


@pytest.mark.parametrize("name,pieces", [("layered", 1), ("in4", 1), ("in5", 1), ("in15", 1), ("in16", 1), ("in62", 1), ("in64", 2),
                                         ("many_inputs", 1), ("long_classes", 2), ("far_apart", 1)])
def test_the_table_that_the_kernel_reads(lib, name, pieces):
    """It says of every class what the plan says; and inputs that are no earlier class, or one too far away, are listed."""
    d = layered(12, 160, 300) if name == "layered" else far_apart() if name == "far_apart" else LISTS[name]()
    p, dep, _, _ = plan_of(lib, d, pieces)
    R, C, row = d.n_recv, len(dep), p["row"].reshape(-1, 16)
    table, listed = p["table"], 0
    assert table.size == 16 * C + p["outputs"].size

    def outputs_are(got, plan):
        got, plan = got.view(np.uint32).astype(np.int64), plan.view(np.uint32).astype(np.int64)
        want = (plan & 0x3ffff) << 2 | (plan & FILL != 0) << 20 | (plan & WIDE != 0) << 21 | plan & (ONLY | LAST)
        return np.array_equal(got, want)

    assert outputs_are(table[16 * C:], p["outputs"])
    words = table[:16 * C].reshape(C, 4, 4)
    assert outputs_are(words[:, :, 1].ravel(), row[:, 4:8].ravel())
    for c in range(C):
        q = words[c]
        short = [(int(q[k & 3, 0]) >> 16 * (k >> 2)) & 0xffff for k in range(8)]
        more = int(q[0, 2])
        x = [c - s if s < 0xc000 else ~(s - 0xc000) for s in short] + p["table_inputs"][(more >> 5) * 4:(more >> 5) * 4 + 4 * (more & 31)].tolist()
        want = inputs_of(row, p, R, c)
        assert [v for v in x if v != ~R] == want, c
        listed += more & 31 != 0 and len(want) <= 8
        assert (more & 31 != 0) == (len(want) > 8 or any(v > c or c - v >= 0xc000 for v in want[:8] if v >= 0)), c
        n = int(row[c, 12])
        assert q[1, 2] == 4 * (16 * C + row[c, 9]) and q[2, 2] == n and q[2, 3] == row[c, 13]
        assert q[0, 3] == row[c, 14] and (n < 1 or q[1, 3] == row[c, 15 if n > 1 else 14])
    assert pieces > 1 or (listed > 0) == (name == "far_apart")      # (a piece may come before what feeds its set)


def two_far_apart():
    """Two graphs of which the ops of one come between those of the other: inputs that are more than the window before what they feed."""
    d = layered(24, 260, 300)
    first, n = d.n_recv, d.n_ops
    new = np.concatenate([np.arange(first), first + (np.arange(n - first) % 2) * ((n - first + 1) // 2) + np.arange(n - first) // 2])
    old = np.argsort(new)
    rows = [np.sort(new[d.col_idx[d.row_ptr[v]:d.row_ptr[v + 1]]]) for v in old]
    return wl.Dag("two_far_apart", n, np.cumsum([0] + [len(r) for r in rows]).astype(np.int32), np.concatenate(rows).astype(np.int32),
                  d.recv_ids, d.op_median, d.recv_bytes)


@pytest.mark.parametrize("name,pieces,by_level", [("layered", 1, False), ("in16", 1, False), ("backwards", 1, True), ("backwards", 2, True),
                                                  ("relabelled", 1, True), ("long_classes", 2, True), ("two_far_apart", 1, True)])
def test_classes_are_numbered_along_the_graph(lib, name, pieces, by_level):
    """As they come where inputs come before what they feed and not far before it, else by level; either way the plan says the same of
    the classes, and the table where their rows and columns are."""
    d = {"layered": lambda: layered(12, 160, 300), "in16": LISTS["in16"], "backwards": lambda: backwards(layered(12, 160, 300)),
         "relabelled": lambda: wl.relabel(layered(12, 160, 300), 5)[0], "long_classes": lambda: backwards(LISTS["long_classes"]()),
         "two_far_apart": two_far_apart}[name]()
    p, dep, cls_of_op, columns = plan_of(lib, d, pieces)
    R, C, row, of = d.n_recv, len(dep), p["row"].reshape(-1, 16), p["cls_of"]
    assert sorted(of) == list(range(C)) and (of.tolist() != list(range(C))) == by_level
    table, order, holds, feeds = p["table"][:16 * C].reshape(C, 4, 4), [j for c in columns for j in c], {}, {}
    assert not table[:, 3, 2:].any()
    for c in range(C):
        x, union = inputs_of(row, p, R, c), 0
        for v in x:
            assert v < c or (not by_level and name == "layered"), (c, v)
            union |= dep[of[v]] if v >= 0 else 1 << ~v
            holds.setdefault(v, []).append(c)
        assert union == dep[of[c]], c
        feeds[c] = sum(v >= 0 for v in x)
        n, first = int(row[c, 12]), int(row[c, 13])
        assert order[first:first + n] == columns[of[c]] and row[c, 14:16].tolist() == (columns[of[c]] + [0, 0])[:2]
        assert table[c, 2, 2] == n and table[c, 2, 3] == first
    assert p["roots"].tolist() == [c for c in range(C) if dep[of[c]] and not feeds[c]]
    assert p["free_cols"].tolist() == [j for c in range(C) if not dep[of[c]] for j in columns[of[c]]]
    for r in range(R):
        assert p["own"][p["own_ptr"][r]:p["own_ptr"][r + 1]].tolist() == holds.get(~r, []), r


def inputs_of(row, p, R, c):
    more = int(row[c, 8])
    at = (more >> 4) * 4
    x = np.concatenate([row[c, :4], p["inputs"][at:at + 4 * (more & 15)]])
    return x[x != ~R].tolist()


@pytest.mark.parametrize("name", ["in65", "q200", "frontier900"])
def test_graphs_without_a_plan(lib, name):
    assert plan_of(lib, LISTS[name](), 1)[0] is None


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
