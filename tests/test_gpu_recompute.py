"""GPU parity of recompute_deps on small graphs.  Building such a handle forms op.dep on the host, so the propagation
kernels (each graph of the parity tests takes another of their forms) run only here: on op.dep cleared before, against the
CPU oracle."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle
from paper_1803_03288_amd import workloads as wl

from test_gpu_parity import SMALL, tt  # noqa: F401


@pytest.mark.parametrize("name", ["tiny", "vgg16", "inception3"] + list(SMALL))
def test_recompute_from_cleared(tt, name):  # noqa: F811
    check(tt, name, SMALL[name]() if name in SMALL else wl.preset(name))


def check(tt, name, d):  # noqa: F811
    want = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    other = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    print(f"[recompute] {name}: n={d.n_ops} R={d.n_recv}", flush=True)
    for k in range(2):
        h.deps_view().zero_()
        h.recompute_deps()
        assert np.array_equal(h.deps().cpu().numpy().view(np.uint64), want), k
    h.deps_view().fill_(-1)
    other.deps_view().zero_()
    tt.recompute_deps_batch([h, other])
    for x in (h, other):
        assert np.array_equal(x.deps().cpu().numpy().view(np.uint64), want)
        x.close()


def wide(levels, width, recvs, fan_in=(2, 3), back=1):
    return wl.layered_dag(31, levels=levels, width=width, fan_in=fan_in, back=back, n_recv=recvs, attach=(1, 3))


# Levels that one pass of the workgroup takes and the level-major kernel does not or just does; about the width from which on the records of
# the chunked one do not fit LDS, with slices of one, two and four words.  w32: rows formed by the kernels in the build.
WIDE = {
    "w1_256": lambda: wide(20, 256, 60), "w1_257": lambda: wide(20, 257, 60), "w1_1024": lambda: wide(18, 1024, 60),
    "w2_288": lambda: wide(20, 288, 128), "w2_289": lambda: wide(20, 289, 128),
    "w4_256": lambda: wide(20, 256, 200), "w4_lists": lambda: wide(20, 256, 200, (4, 9)),
    "w16_257": lambda: wide(20, 257, 1024), "w32_330": lambda: wide(30, 330, 2048), "w32_800": lambda: wide(30, 800, 2000),
    # inputs that have left the ring (8 192 positions with one-word slices)
    "long_w1": lambda: wide(40, 700, 60, back=30), "long_w2": lambda: wide(40, 400, 128, back=30),
}


@pytest.mark.parametrize("name", list(WIDE))
def test_wide_levels(tt, name):  # noqa: F811
    check(tt, name, WIDE[name]())


@pytest.mark.parametrize("name", ["tiny", "inception3", "layered70"])
def test_first_recompute_in_a_captured_graph(tt, name):  # noqa: F811
    """A handle's first recompute_deps, captured, replayed with eager work and cleared rows in between."""
    d = SMALL[name]() if name in SMALL else wl.preset(name)
    want = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rows = h.deps_view()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h.recompute_deps()
    for k in range(4):
        rows.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(rows.cpu().numpy().view(np.uint64), want), k
        if k == 1:
            h.recompute_deps()
    h.close()


def lists_dag(levels, width, recvs):
    """Layered, and every seventh op depends on ops of up to twelve levels before and on more of them than a record holds."""
    rng = np.random.default_rng([levels, width])
    b = wl._Builder()
    rs = [b.recv(1e5) for _ in range(recvs)]
    ops = []
    for lv in range(levels):
        for k in range(width):
            pool = ops[max(0, (lv - (12 if k % 7 == 0 else 2)) * width):]
            preds = [pool[i] for i in rng.choice(len(pool), size=min(len(pool), 9 if k % 7 == 0 else 2), replace=False)] if pool else []
            if lv == 0 or k % 3 == 0:
                preds.append(rs[int(rng.integers(recvs))])
            ops.append(b.op(preds, 1e-3, "op"))
    return b.finish("lists", seed=4, batch=8)


# Slots per level of the kernel with 64-byte slices, a multiple of 32: up to 224 two more waves bring the rows to memory (one to seven per
# thread and level), with 256 there is no room for them; levels just short of and beyond the 32 that are computed in a row.
@pytest.mark.parametrize("levels,width", [(31, 32), (33, 64), (32, 96), (64, 100), (65, 150), (40, 190), (40, 224), (30, 225), (35, 250)])
@pytest.mark.parametrize("kind", ["layered", "lists"])
def test_several_graphs_by_one_launch(tt, levels, width, kind):  # noqa: F811
    d = wide(levels, width, 1024) if kind == "layered" else lists_dag(levels, width, 1000)
    want = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    hs = [tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids) for _ in range(9)]
    for n in (2, 9):
        for h in hs:
            h.deps_view().fill_(-1)
        print(f"[batch] {kind} {levels} x {width}: {n} handles", flush=True)
        tt.recompute_deps_batch(hs[:n])
        for h in hs[:n]:
            assert np.array_equal(h.deps().cpu().numpy().view(np.uint64), want)
    for h in hs:
        h.close()


def lists_at(levels, width, every, back, recvs=1024):
    """Layered, two inputs per op from the level before; every ``every``-th op has nine, from ``back`` levels before."""
    row, col = [0] * (recvs + 1), []
    for v in range(levels * width):
        l, w = divmod(v, width)
        n, at = (9, max(0, l - back)) if v % every == 0 else (2, l - 1)
        col += [v % recvs] if l == 0 else sorted(recvs + at * width + (w + k) % width for k in range(n))
        row.append(len(col))
    n = recvs + levels * width
    return wl.Dag("lists_at", n, np.array(row, np.int32), np.array(col, np.int32), np.arange(recvs, dtype=np.int32), np.ones(levels * width), np.ones(recvs))


# graph, and whether the waves beside those that compute store its rows.  Widths as above; "far": rows that have left the ring, from memory (just
# less than one for a hundred nodes); "near": more than 4 096 list entries, which LDS does not hold; "narrow": rows of eight words, two slices
# to a line; "listed": more from memory
BATCHES = {**{f"w{w}": (lambda l=l, w=w: (wide(l, w, 1024), w <= 224))
              for l, w in ((31, 32), (33, 64), (32, 96), (64, 100), (65, 150), (40, 190), (40, 224), (30, 225))},
           "far": lambda: (lists_at(80, 100, 60, 18), True), "near": lambda: (lists_at(120, 100, 20, 1), True), "narrow": lambda: (lists_at(60, 50, 14, 1, 512), True),
           "listed": lambda: (lists_dag(40, 190, 1000), False), "listed_wide": lambda: (lists_dag(64, 224, 1000), False)}


@pytest.mark.parametrize("name", list(BATCHES))
def test_several_graphs_by_both_kernels(tt, name):  # noqa: F811
    """Batches on either side of the 600 MiB up to which two more waves store the rows.  (Above it some graphs are in the list many
    times: the workgroups that form the same rows write the same words.)"""
    d, _ = BATCHES[name]()
    want = torch.from_numpy(oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids).view(np.int64)).cuda()
    hs = [tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids) for _ in range(5)]
    over = (600 << 20) // (want.numel() * 8) + 1
    for n in (2, 5, over):
        for h in hs:
            h.deps_view().fill_(-1)
        print(f"[batch] {name}: {n} handles", flush=True)
        tt.recompute_deps_batch([hs[i % 5] for i in range(n)])
        for h in hs[:n]:
            assert torch.equal(h.deps_view().view(want.shape), want), (name, n)
    for h in hs:
        h.close()


@pytest.mark.parametrize("name", [n for n in BATCHES if "listed" not in n])
def test_several_graphs_beyond_the_infinity_cache(tt, name):  # noqa: F811
    """Batches just above 256 MiB of rows, formed by a multiple of eight workgroups: through the caches unless lists take longer."""
    d, _ = BATCHES[name]()
    want = torch.from_numpy(oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids).view(np.int64)).cuda()
    hs = [tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids) for _ in range(5)]
    n = ((256 << 20) // (want.numel() * 8) // 8 + 1) * 8
    for h in hs:
        h.deps_view().fill_(-1)
    print(f"[batch] {name}: {n} handles", flush=True)
    tt.recompute_deps_batch([hs[i % 5] for i in range(n)])
    for h in hs:
        assert torch.equal(h.deps_view().view(want.shape), want), name
        h.close()
