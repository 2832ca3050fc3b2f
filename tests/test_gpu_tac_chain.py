"""GPU parity of the chain form of TAC (one lane per sample, large batches of model-shaped graphs): against the
wave-per-sample kernels, which take smaller batches, on every sample, and against the CPU oracle on some of them."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle
from paper_1803_03288_amd import workloads as wl

from helpers import oracle_tac_rows


@pytest.fixture(scope="module")
def tt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1803_03288_amd import binding
    binding.lib()
    return binding


def modules_dag(modules, name="modules"):
    """A chain of modules; a module is a list of branch lengths (layers that read one recv each), joined by an op that
    reads no recv; a length may be zero (a branch of plain ops).  A module of one branch is a piece of a chain."""
    b = wl._Builder()
    x = b.op([], 1e-3, "input")
    for lengths in modules:
        ends = []
        for n in lengths:
            y = b.op([x], 1e-3, "branch")
            for k in range(n):
                y = b.op([y, b.recv(1e5 * (1 + k % 3))], 1e-3, "layer")
                y = b.chain([y], [1e-3] * (k % 3 + 1), "op")
            ends.append(y)
        x = b.op(ends, 1e-3, "join")
    return b.finish(name, seed=5, batch=8)


def overlapping_dag(branches, units, fork=False, name="overlapping"):
    """Units of branches of which neighbours are joined: the recv of a branch in the middle is a sink of two gates.  A layer follows
    every join, and all of them are joined at the end of the unit.  Two branches: the first goes on behind the join, and what it ends
    with is joined with the second too.  fork: two layers follow the layer of every branch in the middle as well."""
    b = wl._Builder()

    def layer(x):
        return b.op([b.op([x, b.recv(1e5 * (1 + len(b.preds) % 3))], 1e-3, "layer")], 1e-3, "op")
    x = b.op([], 1e-3, "input")
    for _ in range(units):
        ends = [layer(x) for _ in range(branches)]
        if branches == 2:
            joins = [b.op(ends, 1e-3, "join"), b.op([layer(ends[0]), ends[1]], 1e-3, "join")]
        else:
            joins = [layer(b.op([y, z], 1e-3, "join")) for y, z in zip(ends, ends[1:])]
            joins += [layer(y) for y in ends[1:-1] for _ in range(2) if fork]
        x = b.op(joins, 1e-3, "join")
    return b.finish(name, seed=5, batch=8)


GRAPHS = {
    "chain": lambda: wl.chain_dag(97),
    "one": lambda: wl.chain_dag(1),
    "two_branches": lambda: modules_dag([[2], [3, 1], [0, 4], [1, 1], [5]]),
    "ends_with_a_join": lambda: modules_dag([[1], [2, 3, 1]]),
    "three_branches": lambda: modules_dag([[3], [1, 2, 9], [4, 4, 4], [1]]),
    "starts_wide": lambda: modules_dag([[2, 1, 3, 2, 1], [1], [2, 2]]),
    "eight_branches": lambda: modules_dag([[1, 2, 3, 1, 2, 3, 1, 2], [2], [1, 1, 1, 1, 1, 1, 1, 1]]),
    "jobs": lambda: wl.independent_jobs_dag(8),
    "resnet50": wl.resnet50_dag,
    # recvs that are sinks of two gates: the kernel's instantiations for two, four and eight slots that know of second gates
    "second_two": lambda: overlapping_dag(2, 12), "second_three": lambda: overlapping_dag(3, 9), "second_four": lambda: overlapping_dag(4, 1),
    "second_five": lambda: overlapping_dag(5, 7), "second_eight": lambda: overlapping_dag(8, 4), "second_fork": lambda: overlapping_dag(3, 6, fork=True),
    "second_fork_four": lambda: overlapping_dag(4, 4, fork=True),
}
SECOND_GATES = {"second_two": 2, "second_three": 4, "second_four": 4, "second_five": 8, "second_eight": 8, "second_fork": 4, "second_fork_four": 8}


def crossed_dag(layers, units, gates, name="crossed"):
    """A chain of layers, and units of a layer and ``gates`` more, which the next layer of the chain joins; with more than one there is a join of
    the first with each of them before, so that its recv is a sink of one gate more than those."""
    b = wl._Builder()

    def layer(*xs):
        return b.chain([b.op([*xs, b.recv(1e5 * (1 + len(b.preds) % 3))], 1e-3, "layer")], [1e-3], "op")
    x = b.op([], 1e-3, "input")
    for _ in range(layers):
        x = layer(x)
    for _ in range(units):
        ends = [layer(x) for _ in range(gates + 1)]
        x = layer(*([b.op([ends[0], y], 1e-3, "join") for y in ends[1:]] if gates > 1 else ends))
    return b.finish(name, seed=5, batch=8)


# every recv is added by one class, as the chain form asks, but: more than eight chains, a recv that is a sink of three gates, 41 gates
REFUSED = {
    "nine": lambda: modules_dag([[30] * 9]), "nine_behind_one": lambda: modules_dag([[200], [8] * 9]), "twelve": lambda: modules_dag([[24] * 12]),
    "sixteen": lambda: modules_dag([[20] * 16]), "three_gates": lambda: crossed_dag(300, 1, 2), "many_gates": lambda: crossed_dag(200, 41, 1),
}


def times(d, B, kind, rng):
    """Timing arrays: lognormal multiples of 2**-30 s; or a few values only, so that most comparisons tie; or with some
    times of zero (which the samples are left to the general kernel for)."""
    if kind == "lognormal":
        op = wl.quantise(1e-3 * np.exp(0.4 * rng.standard_normal((B, d.n_compute))))
        rv = wl.quantise(3e-3 * np.exp(0.6 * rng.standard_normal((B, d.n_recv))))
        return op, rv
    op = wl.QUANTUM * rng.integers(1, 4, size=(B, d.n_compute)).astype(np.float64)
    rv = wl.QUANTUM * rng.integers(2, 7, size=(B, d.n_recv)).astype(np.float64)
    if kind == "zeros":
        rv[rng.random(B) < 0.1, 0] = 0.0
        op[rng.random(B) < 0.1] = 0.0
    return op, rv


@pytest.mark.parametrize("kind", ["lognormal", "ties", "zeros"])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_chain_form(tt, name, kind):
    d = GRAPHS[name]()
    rng = np.random.default_rng([len(name), len(kind)])
    B = 8192 + 64 * 3 + 37
    op, rv = times(d, B, kind, rng)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    print(f"[chain] {name} {kind}: N={d.n_compute} R={d.n_recv} classes={h.n_classes}", flush=True)
    gop, grv = torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda()
    got = tt.tac_simulate(h, gop, grv, want_rank=True)
    torch.cuda.synchronize()
    for lo in range(0, B, 4096):
        part = tt.tac_simulate(h, gop[lo:lo + 4096].contiguous(), grv[lo:lo + 4096].contiguous(), want_rank=True)
        for k in (0, 1, 4, 5, 6, 7, 8):
            assert torch.equal(got[k][lo:lo + 4096], part[k]), (name, kind, lo, k)
    rows = sorted(set(np.linspace(0, B - 1, 12 if d.n_recv > 100 else 60).astype(int).tolist()))
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    eo = oracle.tac(dep, d.recv_ids, op[rows], rv[rows])[0]
    assert np.array_equal(got[0][rows].cpu().numpy(), eo)
    em = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, eo, op[rows], rv[rows])
    for k in range(5):
        np.testing.assert_allclose(got[4 + k][rows].cpu().numpy(), em[k], rtol=1e-12, atol=0)
    # the orders alone, and the same samples stored as float32 (exact for the small multiples)
    only = tt.tac_priority(h, gop, grv, want_rank=False)[0]
    assert torch.equal(only, got[0])
    if kind != "lognormal":
        f32 = tt.tac_simulate(h, gop.float(), grv.float())
        assert torch.equal(f32[0], got[0]) and torch.equal(f32[4], got[4])


def test_chain_form_inception(tt):
    """Seven class slots per lane: the chain form from 64 samples on, whose results are those of single samples."""
    d = wl.inception3_dag()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    for B in (64, 65, 200):
        op, rv = wl.timing_samples(d, 0, B)
        gop, grv = torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda()
        got = tt.tac_simulate(h, gop, grv, want_rank=True)
        for lo in range(0, B, 63):
            part = tt.tac_simulate(h, gop[lo:lo + 63].contiguous(), grv[lo:lo + 63].contiguous(), want_rank=True)
            for k in (0, 1, 4, 5, 6, 7, 8):
                assert torch.equal(got[k][lo:lo + 63], part[k])
    rows = [0, 63, 64, 199]
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    eo, er = oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[:2]
    assert np.array_equal(got[0][rows].cpu().numpy(), eo) and np.array_equal(got[1][rows].cpu().numpy(), er)


@pytest.mark.parametrize("name", list(REFUSED))
def test_graphs_without_the_form(tt, name):
    """First and second call of a batch large enough for the chain form, on a graph that has more chains or gates than it takes."""
    d = REFUSED[name]()
    rng = np.random.default_rng(len(name))
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    assert h.n_classes > 256                                  # (from 64 samples on)
    print(f"[chain] {name}: N={d.n_compute} R={d.n_recv} classes={h.n_classes}", flush=True)
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    for B in (64, 70):
        op, rv = times(d, B, "lognormal", rng)
        got = tt.tac_simulate(h, torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda(), want_rank=True)
        rows = [0, 33, B - 1]
        eo, er = oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[:2]
        assert np.array_equal(got[0][rows].cpu().numpy(), eo) and np.array_equal(got[1][rows].cpu().numpy(), er)
        em = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, eo, op[rows], rv[rows])
        for k in range(5):
            np.testing.assert_allclose(got[4 + k][rows].cpu().numpy(), em[k], rtol=1e-12, atol=0)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_totals_past_the_caches(dtype):
    """A batch whose rows and totals exceed 432 MiB writes the totals past the caches; parts of it do not.  Times are
    multiples of 2^-20 below 2^-6, so every sum is exact and the bytes are the same."""
    import torch
    from paper_1803_03288_amd import binding as tt, workloads as wl
    d = wl.resnet50_dag()
    gen = torch.Generator(device="cuda").manual_seed(5)
    B, part, n_comp = 65536, 16387, d.n_ops - d.n_recv
    op = (torch.randint(1, 1 << 14, (B, n_comp), device="cuda", generator=gen) * 2.0 ** -20).to(getattr(torch, dtype))
    rv = (torch.randint(1, 1 << 14, (B, d.n_recv), device="cuda", generator=gen) * 2.0 ** -20).to(getattr(torch, dtype))
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    whole = tt.tac_simulate(h, op, rv)
    for b in range(0, B, part):
        for x, y in zip(whole, tt.tac_simulate(h, op[b:b + part].contiguous(), rv[b:b + part].contiguous())):
            assert (x is None and y is None) or torch.equal(x[b:b + part], y)
