"""GPU parity of the iteration with send ops where a lane follows a sample: the straight form (samples whose ops run by
ascending id) with the samples it gives up, and the event-driven form: several lanes and waves per compute unit, batches
that leave lanes without a sample, counters of half a byte and of a byte, ops past the first summary word, sends without
predecessors, and the graphs that stay with the wave-per-sample form.  Against the CPU oracle, exact on quantised times."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle
from paper_1803_03288_amd import workloads as wl

from test_gpu_sends import GRAPHS, compare, cuda, leaves_of, tt, with_sends  # noqa: F401


def fan_in(k):
    """k jobs of a recv and an op, all joined by one op, which two sends follow; one more send has no predecessor."""
    n = 2 * k + 4
    pred = {k + i: [i] for i in range(k)}
    pred[2 * k] = list(range(k, 2 * k))
    pred[2 * k + 1] = pred[2 * k + 2] = [2 * k]
    row_ptr, col = np.zeros(n + 1, dtype=np.int32), []
    for v in range(n):
        col += pred.get(v, [])
        row_ptr[v + 1] = len(col)
    d = wl.Dag("fan_in", n, row_ptr, np.array(col, dtype=np.int32), np.arange(k, dtype=np.int32), np.ones(n - k), np.ones(k))
    return d, np.array([2 * k + 1, 2 * k + 2, 2 * k + 3], dtype=np.int32)


MORE = {
    "fan_in15": lambda: fan_in(15),         # counters of half a byte
    "fan_in16": lambda: fan_in(16),         # of a byte
    "fan_in255": lambda: fan_in(255),
    "fan_in256": lambda: fan_in(256),       # stays with the wave-per-sample form
    "vgg16": lambda: with_sends(wl.preset("vgg16"), 32, 7),
    "long_chain": lambda: with_sends(wl.chain_dag(300), 30, 9),             # straight: every op waits alone
    "funnel32": lambda: with_sends(wl.funnel_dag(32, 250), 20, 10),         # an op with a tile's worth of recvs
    "funnel33": lambda: with_sends(wl.funnel_dag(33, 250), 20, 11),
    "relabelled": lambda: (lambda d: (d, leaves_of(d)))(                    # ids in no topological order
        wl.relabel(wl.layered_dag(33, levels=30, width=9, fan_in=(1, 3), back=3, n_recv=60, attach=(1, 3)), 5)[0]),
    "layered270": lambda: with_sends(                                       # hardly a sample goes straight
        wl.layered_dag(34, levels=30, width=9, fan_in=(1, 3), back=3, n_recv=60, attach=(1, 3)), 60, 12),
    "no_recv": lambda: with_sends(wl.no_recv_dag(17), 5, 8),
}


@pytest.mark.parametrize("name,B", [(g, B) for g in list(MORE) + ["tiny", "layered", "wide_fanout"] for B in (1, 257, 4200)] +
                         [("resnet50", 2100), ("inception3", 600)])
def test_sends_by_lanes(tt, name, B):  # noqa: F811
    d, sends = (MORE.get(name) or GRAPHS[name])()
    R = d.n_recv
    rng = np.random.default_rng(B)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    op = rng.integers(0, 2000, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(0, 4000, size=(B, R)).astype(np.float64) * wl.QUANTUM
    orders = np.argsort(rng.random((B, R)), axis=1).astype(np.int32)
    print(f"[sends] {name}: n={d.n_ops} R={R} sends={sends.size} B={B}", flush=True)
    gop, grv = cuda(op), cuda(rv)
    for order in (orders, orders[0]):
        compare(tt.simulate_sends(h, sends, cuda(order), gop, grv),
                oracle.simulate_sends(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, sends, order, op, rv), True, f"{name} {B}")
    h.close()
