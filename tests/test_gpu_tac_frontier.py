"""GPU parity of TAC by the frontier form (graphs with more than 1 024 classes, batches of more than two samples per compute
unit): where its lists and records change shape, and where samples outgrow its lists and are left to the bit-sliced kernel,
against the CPU oracle."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle
from paper_1803_03288_amd import workloads as wl

from helpers import oracle_tac_rows

B = 521                                     # (more than two samples on each of 256 compute units)


@pytest.fixture(scope="module")
def tt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1803_03288_amd import binding
    binding.lib()
    assert torch.cuda.get_device_properties(0).multi_processor_count * 2 < B
    return binding


def layered(levels, width, recvs, fan_in=(1, 4), attach=(1, 8)):
    return wl.layered_dag(43, levels=levels, width=width, fan_in=fan_in, back=3, n_recv=recvs, attach=attach)


def with_layers(first, recvs):
    """``first(builder, recvs)`` in front of layers of ops over the same recvs, which bring 1 024 classes and more."""
    b = wl._Builder()
    rs = [b.recv(1e5 * (1 + k % 7)) for k in range(recvs)]
    above = first(b, rs)
    g = np.random.default_rng(6)
    for level in range(24):
        below = [b.op([above[i] for i in g.choice(len(above), size=min(len(above), 2), replace=False)] +
                      [rs[i] for i in g.choice(recvs, size=1 + (level % 2), replace=False)], 1e-3, "op") for _ in range(90)]
        above = below
    return b.finish("layers", seed=3, batch=4)


def fans(n_in):
    """Ops with n_in inputs, classes that point or do not by then, and n_in outputs of one class."""
    def first(b, rs):
        heads = [b.op([rs[i], rs[(i + i % 3) % len(rs)]], 1e-3, "op") for i in range(n_in)]
        wide = [b.op(heads, 1e-3, "op"), b.op(heads + rs[:3], 1e-3, "op")]
        return wide + [b.op([wide[0], rs[i]], 1e-3, "op") for i in range(n_in)]
    return with_layers(first, 320)


def many_pointed(k):
    """As soon as recv 0 has been transferred k recvs have P > 0: more than the kernel's Q holds, or just as many."""
    return with_layers(lambda b, rs: [b.op([rs[0], rs[1 + i]], 1e-3, "op") for i in range(k)], 300)


def long_frontier(k):
    """k classes with two outstanding recvs each behind one that points at a third."""
    def first(b, rs):
        a = b.op([rs[0]], 1e-3, "op")
        return [b.op([a, rs[1 + i % 290], rs[1 + (i + 1 + i // 290) % 290]], 1e-3, "op") for i in range(k)]
    return with_layers(first, 300)


def frontier_in_two(k):
    """A frontier of 290 classes from the start and k more once recv 0 has been transferred, fewer at a time than the stack holds."""
    def first(b, rs):
        a = b.op([rs[0]], 1e-3, "op")
        return [b.op([rs[1 + i], rs[1 + (i + 1) % 290]], 1e-3, "op") for i in range(290)] + \
            [b.op([a, rs[1 + i], rs[1 + (i + 2) % 290]], 1e-3, "op") for i in range(k)]
    return with_layers(first, 300)


def long_classes():
    """Classes of up to 700 ops: split into pieces, more than two columns each."""
    def first(b, rs):
        out = []
        for i in range(8):
            x = b.op([rs[i], rs[i + 1]], 1e-4, "op")
            for _ in range(2 + 100 * i):
                x = b.op([x], 1e-4, "op")
            out.append(x)
        b.op([], 1e-3, "op")                # (depends on no recv)
        return out
    return with_layers(first, 320)


def backwards(d):
    """The same graph with its ops numbered the other way round: no input of a class is an earlier class, as they come."""
    rows = [(d.n_ops - 1 - d.col_idx[d.row_ptr[v]:d.row_ptr[v + 1]])[::-1] for v in range(d.n_ops)][::-1]
    return wl.Dag(name="backwards", n_ops=d.n_ops, row_ptr=np.cumsum([0] + [len(r) for r in rows]).astype(np.int32),
                  col_idx=np.concatenate(rows).astype(np.int32), recv_ids=(d.n_ops - 1 - d.recv_ids)[::-1].astype(np.int32).copy(),
                  op_median=d.op_median[::-1].copy(), recv_bytes=d.recv_bytes[::-1].copy())


GRAPHS = {
    "layered": lambda: layered(40, 40, 400),
    "one_word": lambda: layered(40, 150, 63, attach=(1, 4)),
    "word_edge": lambda: layered(40, 100, 128, attach=(2, 4)),
    "many_inputs": lambda: layered(30, 90, 500, fan_in=(1, 24)),            # up to four, up to fifteen and more inputs
    "own_recvs": lambda: layered(30, 60, 500, attach=(8, 16)),             # more than eight outstanding recvs
    "in4": lambda: fans(4), "in5": lambda: fans(5), "in15": lambda: fans(15), "in16": lambda: fans(16),
    "in61": lambda: fans(61),
    "in62": lambda: fans(62), "in64": lambda: fans(64),
    "in65": lambda: fans(65),               # more inputs than the form takes: the bit-sliced kernel
    "q127": lambda: many_pointed(127), "q200": lambda: many_pointed(200),
    "frontier400": lambda: long_frontier(400), "frontier900": lambda: long_frontier(900),
    # a little longer than the lists: the plan takes the form, the kernel leaves samples
    "q140": lambda: many_pointed(140), "frontier300": lambda: long_frontier(300), "frontier500": lambda: frontier_in_two(210),
    "long_classes": long_classes,
    # ids that do not rise along the graph: classes numbered by level
    "fallen": lambda: backwards(layered(40, 40, 400)), "fallen_own": lambda: backwards(layered(30, 60, 500, attach=(8, 16))),
    "fallen_long": lambda: backwards(long_classes()), "fallen_in64": lambda: backwards(fans(64)),
    "relabelled": lambda: wl.relabel(layered(40, 100, 300), 3)[0],
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_tac_by_the_frontier_form(tt, name):
    d = GRAPHS[name]()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    assert h.n_classes > 1024, h.n_classes
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rng = np.random.default_rng(7)
    rows = [0, 255, B - 1]

    def ints(lo, hi, n):
        return rng.integers(lo, hi, size=(B, n)).astype(np.float64) * wl.QUANTUM

    zero = ints(1, 1 << 20, d.n_recv)
    zero[::5, 1] = 0.0                      # (these go to the general kernel, between the others)
    cases = [("distinct", ints(1, 1 << 20, d.n_compute), ints(1, 1 << 20, d.n_recv)),
             ("ties", ints(0, 3, d.n_compute), ints(1, 4, d.n_recv)),
             ("zeros", ints(0, 1 << 20, d.n_compute), zero),
             ("lognormal", rng.lognormal(-7.0, 0.5, size=(B, d.n_compute)), rng.lognormal(-6.5, 1.5, size=(B, d.n_recv)))]
    for what, op, rv in cases:
        print(f"[frontier] {name} {what}: classes={h.n_classes} R={d.n_recv}", flush=True)
        got = tt.tac_simulate(h, torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda(), want_rank=True)
        eo, er = oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[:2]
        assert np.array_equal(got[0].cpu().numpy()[rows], eo), what
        assert np.array_equal(got[1].cpu().numpy()[rows], er), what
        order = np.sort(got[0].cpu().numpy(), axis=1)
        assert (order == np.arange(d.n_recv)).all()
        exp = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, eo, op[rows], rv[rows])
        # sums of at most n_ops float64 terms, in another order; E and S lose what U - m, U - L cancel
        rtol = d.n_ops * 2.0 ** -53
        m, E, U, L, S = (x.cpu().numpy()[rows] for x in got[4:9])
        em, eE, eU, eL, eS = exp
        for g, e in ((m, em), (U, eU), (L, eL)):
            np.testing.assert_allclose(g, e, rtol=rtol, atol=0)
        np.testing.assert_allclose(E, eE, rtol=0, atol=4 * rtol * float((eU / (eU - eL)).max()))
        np.testing.assert_allclose(S, eS, rtol=0, atol=4 * rtol * float((eU / eL).max()))
        again = tt.tac_simulate(h, torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda(), want_rank=True)
        for k in (0, 1, 4, 5, 6, 7, 8):
            assert torch.equal(got[k], again[k]), (what, k)
    # a batch for the bit-sliced kernel gives the same; float32 storage of values that float32 holds as well
    op, rv = cases[0][1], cases[0][2]
    full = tt.tac_simulate(h, torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda(), want_rank=True)
    part = tt.tac_simulate(h, torch.from_numpy(op[:97]).cuda(), torch.from_numpy(rv[:97]).cuda(), want_rank=True)
    f32 = tt.tac_simulate(h, torch.from_numpy(op).cuda().float(), torch.from_numpy(rv).cuda().float(), want_rank=True)
    for k in (0, 1, 4, 5, 6, 7, 8):
        assert torch.equal(full[k][:97], part[k]), k
        assert torch.equal(full[k], f32[k]), k
    h.close()


# states in LDS and in memory; the last two: samples are left to the bit-sliced kernel, their lists full
@pytest.mark.parametrize("name,many", [("layered", 8200), ("many_inputs", 12001), ("q140", 8200), ("frontier500", 12001)])
def test_several_samples_per_wave(tt, name, many):
    """More samples than there are waves at a time: what a wave has of the one before it is not seen in the next."""
    d = GRAPHS[name]()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rng = np.random.default_rng(8)
    op = rng.integers(1, 1 << 20, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(1, 1 << 20, size=(B, d.n_recv)).astype(np.float64) * wl.QUANTUM
    op[1::4], rv[1::4] = np.floor(op[1::4] / wl.QUANTUM % 3) * wl.QUANTUM, np.floor(rv[1::4] / wl.QUANTUM % 3 + 1) * wl.QUANTUM      # (ties)
    op[2::4], rv[2::4] = rng.exponential(1e-3, size=op[2::4].shape), rng.lognormal(-6.5, 1.5, size=rv[2::4].shape)
    rv[3::8, 2] = 0.0
    print(f"[frontier] {name}: classes={h.n_classes} R={d.n_recv} B={many}", flush=True)
    op, rv = torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda()
    first = tt.tac_simulate(h, op, rv, want_rank=True)
    rows = [0, 1, 3, 4, B - 1]
    eo = oracle_tac_rows(dep, d.recv_ids, op.cpu().numpy()[rows], rv.cpu().numpy()[rows])[0]
    assert np.array_equal(first[0].cpu().numpy()[rows], eo)
    of = torch.arange(many, device="cuda") % B
    got = tt.tac_simulate(h, op[of], rv[of], want_rank=True)
    for k in (0, 1, 4, 5, 6, 7, 8):
        assert torch.equal(got[k], first[k][of]), k
    h.close()


def side_by_side(parts):
    """Graphs that have nothing to do with each other, one after the other: samples are busy in all of them, thousands of classes apart."""
    n = np.cumsum([0] + [d.n_ops for d in parts])
    edges = np.cumsum([0] + [d.row_ptr[-1] for d in parts])
    return wl.Dag(name="side_by_side", n_ops=int(n[-1]),
                  row_ptr=np.concatenate([d.row_ptr[:-1] + e for d, e in zip(parts, edges)] + [edges[-1:]]).astype(np.int32),
                  col_idx=np.concatenate([d.col_idx + k for d, k in zip(parts, n)]).astype(np.int32),
                  recv_ids=np.concatenate([d.recv_ids + k for d, k in zip(parts, n)]).astype(np.int32),
                  op_median=np.concatenate([d.op_median for d in parts]), recv_bytes=np.concatenate([d.recv_bytes for d in parts]))


# The counters in LDS are those of 4 096 classes: some more, classes busy in several places, all of them moving the other way.
@pytest.mark.parametrize("name", ["layers", "three", "fans", "backwards"])
def test_counters_in_and_out_of_the_window(tt, name):
    d = {"layers": lambda: layered(70, 110, 500), "three": lambda: side_by_side([layered(30, 90, 120), layered(32, 100, 150), layered(31, 95, 90)]),
         "fans": lambda: side_by_side([fans(16), layered(36, 110, 200), fans(9)]), "backwards": lambda: backwards(layered(70, 110, 500))}[name]()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    assert h.n_classes > 4096, h.n_classes
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rng = np.random.default_rng(9)
    op = rng.integers(1, 1 << 20, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(1, 1 << 20, size=(B, d.n_recv)).astype(np.float64) * wl.QUANTUM
    rv[1::2, :d.n_recv // 2] *= 64.0        # (the classes that come first are done last)
    print(f"[frontier] {name}: classes={h.n_classes} R={d.n_recv}", flush=True)
    got = tt.tac_simulate(h, torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda(), want_rank=True)
    rows = [0, 1, B - 1]
    assert np.array_equal(got[0].cpu().numpy()[rows], oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[0])
    part = tt.tac_simulate(h, torch.from_numpy(op[:97]).cuda(), torch.from_numpy(rv[:97]).cuda(), want_rank=True)       # bit-sliced
    for k in (0, 1, 4, 5, 6, 7, 8):
        assert torch.equal(got[k][:97], part[k]), k
    h.close()
