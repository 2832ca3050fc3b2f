"""GPU parity of the class totals that four lanes with one class add together (TAC in registers of five to eight class slots per
lane, several channels and simulation with an order each with more than four): runs of columns of one class at every offset from the sixteen columns that four
lanes take, classes that come back within them, rows that end anywhere in them; against the CPU oracle.  The simulations add that way where
runs are long (far_...), else lane by lane."""

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


def runs(recvs, lengths, tail=0, back=0):
    """One class per recv, its ops in a row: ``lengths`` of them, round robin; then ``tail`` ops of the last class and, for the
    first ``back`` classes, two ops each by turns (A B A B)."""
    b = wl._Builder()
    rs = [b.recv(1e5 * (1 + k % 7)) for k in range(recvs)]
    last = []
    for i, r in enumerate(rs):
        last.append(r)
        for _ in range(lengths[i % len(lengths)]):
            last[i] = b.op([last[i]], 1e-4, "op")
    for _ in range(tail):
        last[-1] = b.op([last[-1]], 1e-4, "op")
    for i in range(0, back, 2):
        for k in (i, i + 1, i, i + 1):
            last[k] = b.op([last[k]], 1e-4, "op")
    return b.finish("runs", seed=3, batch=4)


GRAPHS = {
    "whole_quads": lambda: runs(290, [16]),                     # every four lanes one class, the last tile not full
    "offsets": lambda: runs(290, [13, 17, 16, 31, 1, 5]),
    "long": lambda: runs(300, [1] * 29 + [700]),                # classes over several tiles of 256 columns
    "short": lambda: runs(330, [1, 2, 3]),                      # no four lanes with one class
    "back": lambda: runs(300, [15, 16], back=40),
    "six_slots": lambda: runs(380, [16, 14]),
    "eight_slots": lambda: runs(480, [12, 17]),
    # runs long enough that the simulations add by quads too
    "far": lambda: runs(290, [48]),
    "far_offsets": lambda: runs(300, [45, 61, 3, 52, 64]),
    "far_six_slots": lambda: runs(370, [48, 50, 33, 1]),
    "far_seven_slots": lambda: runs(400, [46, 19, 71]),
    "far_eight_slots": lambda: runs(450, [65, 2, 43]),
    **{f"far_tail{k}": (lambda k=k: runs(288, [60], tail=k)) for k in (1, 3, 253, 255)},
    **{f"tail{k}": (lambda k=k: runs(288, [16], tail=k)) for k in (1, 2, 3, 4, 253, 255, 256, 257)},
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_class_totals_of_runs(tt, name):
    d = GRAPHS[name]()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    assert 256 < h.n_classes <= 512, h.n_classes
    rng = np.random.default_rng(11)
    B = 9
    # whole multiples of 2^-30 s: every sum is exact, in any order
    op = rng.integers(0, 1 << 20, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(1, 1 << 20, size=(B, d.n_recv)).astype(np.float64) * wl.QUANTUM
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    eo, er = oracle_tac_rows(dep, d.recv_ids, op, rv)[:2]
    exp = oracle.simulate(*args, eo, op, rv)
    orders = np.stack([rng.permutation(d.n_recv) for _ in range(B)]).astype(np.int32)
    chan = (np.arange(d.n_recv) % 3).astype(np.int32)
    for dtype in (np.float64, np.float32):
        # (20 bits and fewer fit a float32)
        gop, grv = torch.from_numpy(op.astype(dtype)).cuda(), torch.from_numpy(rv.astype(dtype)).cuda()
        print(f"[totals] {name} {np.dtype(dtype).name}: N={d.n_compute} classes={h.n_classes}", flush=True)
        got = tt.tac_simulate(h, gop, grv, want_rank=True)
        assert np.array_equal(got[0].cpu().numpy(), eo)
        assert np.array_equal(got[1].cpu().numpy(), er)
        for a, b, what in zip(got[4:9], exp, "mEULS"):
            assert np.array_equal(a.cpu().numpy(), b), what
        alone = tt.simulate(h, torch.from_numpy(orders).cuda(), gop, grv)
        for a, b, what in zip(alone, oracle.simulate(*args, orders, op, rv), "mEULS"):
            assert np.array_equal(a.cpu().numpy(), b), what
        # (above 1 024 samples the simulation adds by quads where runs are long: the same samples again and again)
        again = tt.simulate(h, *(torch.from_numpy(x).cuda().repeat(115, 1) for x in (orders, op.astype(dtype), rv.astype(dtype))))
        for a, b, what in zip(again, alone, "mEULS"):
            assert torch.equal(a, b.repeat(115)), what
        if dtype == np.float64:
            many = tt.simulate_channels(h, 3, chan, torch.from_numpy(orders).cuda(), gop, grv)
            for a, b, what in zip(many, oracle.simulate_channels(*args, 3, chan, orders, op, rv), "mEULS"):
                assert np.array_equal(a.cpu().numpy(), b), what


@pytest.mark.parametrize("recvs", [1, 2, 3, 4, 5, 63, 64, 65, 255, 256, 257, 511, 512])
def test_an_order_each(tt, recvs):
    """The simulation with an order each, whose positions share their place with times and sums: every remainder of four recvs, where
    the levels of the maxima grow, the most recvs it takes."""
    # rows of one run, of one to all recvs
    b = wl._Builder()
    rs = [b.recv(1e5 * (1 + k % 7)) for k in range(recvs)]
    for i in range(recvs):
        for _ in range(1 + i % 3):
            b.op(rs[i:i + 1 + (7 * i) % recvs], 1e-4, "op")
    d = b.finish("spans", seed=3, batch=4)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rng = np.random.default_rng(recvs)
    B = 700
    op = rng.integers(0, 1 << 20, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(0, 1 << 20, size=(B, d.n_recv)).astype(np.float64) * wl.QUANTUM
    orders = np.stack([rng.permutation(recvs) for _ in range(B)]).astype(np.int32)
    rows = np.r_[0:12, B - 12:B]
    exp = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, orders[rows], op[rows], rv[rows])
    for dtype in (np.float64, np.float32):
        print(f"[an order each] {recvs} {np.dtype(dtype).name}: N={d.n_compute} classes={h.n_classes}", flush=True)
        got = tt.simulate(h, torch.from_numpy(orders).cuda(), torch.from_numpy(op.astype(dtype)).cuda(),
                          torch.from_numpy(rv.astype(dtype)).cuda())
        for a, b_, what in zip(got, exp, "mEULS"):
            assert np.array_equal(a.cpu().numpy()[rows], b_), what
