"""The one-lane-per-sample forms (TAC by chains, simulation, iteration with sends: straight and event-driven) on times that
are not quantised, so that sums in another order round differently: against the CPU oracle within what float64 gives.

A sum of n positive float64 terms in any order is off by at most n u of itself, u = 2**-53; makespan, U and L are sums and
maxima of sums of the n = N + R times of a sample, so two correct results differ by at most 2 n u of themselves.  In
E = (U - m) / (U - L) numerator and denominator are each off by up to 2 n u U, so two results differ by at most
8 n u U / (U - L) (0 <= E <= 1); likewise S = (U - L) / L by at most 8 n u (1 + S)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle
from paper_1803_03288_amd import workloads as wl

from helpers import tac_order_up_to_near_ties
from test_gpu_sends import leaves_of, with_sends
from test_gpu_sim_lanes import GRAPHS as LANE_GRAPHS
from test_gpu_tac_chain import GRAPHS as CHAIN_GRAPHS
from test_gpu_tac_chain import tt  # noqa: F401

ROWS = 48       # different samples; a larger batch repeats them


def draw(d, seed, recv_scale=2e-3, long_ops=False):
    rng = np.random.default_rng(seed)
    op = rng.lognormal(np.log(1e-3), 0.5, size=(ROWS, d.n_compute))
    rv = rng.lognormal(np.log(recv_scale), 0.7, size=(ROWS, d.n_recv))
    if long_ops:
        op[rng.random(op.shape) < 0.1] *= 1e4       # long ops between short ones
    return op, rv, rng


def batch(a, B):
    return torch.from_numpy(a).cuda().repeat((B + ROWS - 1) // ROWS, 1)[:B].contiguous()


def same_for_every_copy(got, what):
    for x in got:
        if x is not None:
            for lo in range(ROWS, x.shape[0], ROWS):
                assert torch.equal(x[lo:lo + ROWS], x[:x.shape[0] - lo][:ROWS]), (what, lo)


def close(got, exp, n, what):
    u = 2.0 ** -53
    m, E, U, L, S = exp
    bound = (2 * n * u * m, 8 * n * u * U / (U - L), 2 * n * u * U, 2 * n * u * L, 8 * n * u * (1 + S))
    for a, b, t, nm in zip(got, exp, bound, "m E U L S".split()):
        diff = np.abs(a[:ROWS].cpu().numpy() - b)
        assert (diff <= t).all(), f"{what} {nm}: {float((diff / t).max())} times the bound"


@pytest.mark.parametrize("name,B", [("chain", 8192 + 65), ("two_branches", 8192 + 65), ("three_branches", 8192 + 65), ("jobs", 8192 + 65),
                                    ("resnet50", 8192 + 65), ("inception3", 130)])
def test_tac_by_chains(tt, name, B):  # noqa: F811
    d = wl.inception3_dag() if name == "inception3" else CHAIN_GRAPHS[name]()
    op, rv, _ = draw(d, 41)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    print(f"[unquantised] chains {name}: N={d.n_compute} R={d.n_recv}", flush=True)
    got = tt.tac_simulate(h, batch(op, B), batch(rv, B), want_rank=True)
    same_for_every_copy(got, name)
    order = got[0][:ROWS].cpu().numpy()
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rows = range(0, ROWS, 16) if name == "inception3" else range(0, ROWS, 4)
    near = [tac_order_up_to_near_ties(oracle, d, dep, op[b], rv[b], order[b]) for b in rows]
    print(f"[unquantised] near ties per sample: {near}", flush=True)
    close(got[4:], oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, order, op, rv), d.n_ops, name)


@pytest.mark.parametrize("name", ["tiny", "vgg16", "layered", "chain128"])
def test_simulation_by_lanes(tt, name):  # noqa: F811
    d = LANE_GRAPHS[name]()
    op, rv, rng = draw(d, 42)
    orders = np.argsort(rng.random((ROWS, d.n_recv)), axis=1).astype(np.int32)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    print(f"[unquantised] lanes {name}: N={d.n_compute} R={d.n_recv}", flush=True)
    for dtype in (np.float64, np.float32):
        o, r = op.astype(dtype), rv.astype(dtype)
        for order, B in ((orders[0], 3 * ROWS + 5), (orders, 24 * 1024 + 29)):
            given = torch.from_numpy(order).cuda() if order.ndim == 1 else batch(order, B)
            got = tt.simulate(h, given, batch(o, B), batch(r, B))
            same_for_every_copy(got, name)
            exp = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, order, o.astype(np.float64), r.astype(np.float64))
            close(got, exp, d.n_ops, f"{name} {dtype.__name__} {order.ndim}")


SENDS = {
    "resnet50": lambda: with_sends(wl.preset("resnet50"), 161, 5),
    "vgg16": lambda: with_sends(wl.preset("vgg16"), 32, 7),
    "long_chain": lambda: with_sends(wl.chain_dag(300), 30, 9),
    "layered": lambda: (lambda d: (d, leaves_of(d)))(
        wl.layered_dag(31, levels=7, width=9, fan_in=(1, 3), back=3, n_recv=20, attach=(1, 3))),
}


@pytest.mark.parametrize("long_ops", [False, True])
@pytest.mark.parametrize("name", list(SENDS))
def test_sends(tt, name, long_ops):  # noqa: F811
    d, sends = SENDS[name]()
    # (transfers that run ahead, as a deployed order's do: the straight form; random orders: many samples given up)
    op, rv, rng = draw(d, 43, recv_scale=2e-4, long_ops=long_ops)
    orders = np.argsort(rng.random((ROWS, d.n_recv)), axis=1).astype(np.int32)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    print(f"[unquantised] sends {name}: n={d.n_ops} R={d.n_recv} sends={sends.size}", flush=True)
    B = 2100
    for order in (np.arange(d.n_recv, dtype=np.int32), orders):
        given = torch.from_numpy(order).cuda() if order.ndim == 1 else batch(order, B)
        got = tt.simulate_sends(h, sends, given, batch(op, B), batch(rv, B))
        same_for_every_copy(got, name)
        exp = oracle.simulate_sends(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, sends, order, op, rv)
        close(got, exp, d.n_ops, f"{name} {order.ndim}")
