"""GPU parity where the work of a wave changes its layout: consecutive positions and classes per lane (several channels, the
order search), where the release positions of classes come from (one order for a sample each) and the class slots, tables and waves of TAC in registers, against the CPU oracle."""

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


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def layered(levels, width, recvs, attach=(1, 8)):
    return wl.layered_dag(17, levels=levels, width=width, fan_in=(1, 4), back=3, n_recv=recvs, attach=attach)


def chain(recvs, free=0):
    """A class per recv, rows of one run."""
    b = wl._Builder()
    rs = [b.recv(1e5 * (1 + k % 7)) for k in range(recvs)]
    x = []
    for r in rs:
        x = [b.op(x + [r], 1e-3, "op")]
    for _ in range(free):
        b.op([], 1e-3, "op")                # (depends on no recv)
    return b.finish("chain", seed=3, batch=4)


# recvs on both sides of every 64 of a wave's positions per lane; rows of one run and of many
POSITIONS = {f"chain{r}": (lambda r=r: chain(r, r % 3 if r < 511 else 0)) for r in (1, 2, 63, 64, 65, 192, 193, 319, 320, 321, 448, 511, 512)}
POSITIONS.update({f"layered{r}": (lambda r=r: layered(9, 9, r, (1, 5))) for r in (3, 64, 128, 257, 449, 512)})
POSITIONS.update({f"many_classes{r}": (lambda r=r: layered(24, 18, r, (2, 6))) for r in (6, 15, 16, 17, 28, 130, 300)})


@pytest.mark.parametrize("name", list(POSITIONS))
def test_consecutive_positions(tt, name):
    d = POSITIONS[name]()
    R, B = d.n_recv, 23
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(*args)
    rng = np.random.default_rng(5)
    orders = np.stack([rng.permutation(R) for _ in range(B)]).astype(np.int32)
    op = rng.integers(0, 50, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM      # (equal and zero times as well)
    rv = rng.integers(0, 50, size=(B, R)).astype(np.float64) * wl.QUANTUM
    for n_ch in (1, 3, 64):
        chan = rng.integers(0, n_ch, size=R).astype(np.int32)
        exp = oracle.simulate_channels(*args, n_ch, chan, orders, op, rv)
        got = tt.simulate_channels(h, n_ch, chan, cuda(orders), cuda(op), cuda(rv))
        for g, e in zip(got, exp):
            assert np.array_equal(g.cpu().numpy(), e), n_ch
        exp1 = oracle.simulate_channels(*args, n_ch, chan, orders[0], op, rv)
        got1 = tt.simulate_channels(h, n_ch, chan, cuda(orders[0]), cuda(op), cuda(rv))
        assert np.array_equal(got1[0].cpu().numpy(), exp1[0])
    h.check_orders()
    exp = oracle.simulate(*args, orders, op, rv)
    for g, e in zip(tt.simulate(h, cuda(orders), cuda(op), cuda(rv)), exp):
        assert np.array_equal(g.cpu().numpy(), e)
    exp = oracle.simulate(*args, orders[0], op, rv)
    for g, e in zip(tt.simulate(h, cuda(orders[0]), cuda(op), cuda(rv)), exp):
        assert np.array_equal(g.cpu().numpy(), e)
    h.check_orders()
    if h.n_classes <= 512:
        moves = rng.integers(0, R, size=(64, 2)).astype(np.int32)
        exp = oracle.order_search(*args, orders, moves, op, rv)
        for g, e in zip(tt.order_search(h, cuda(orders), cuda(moves), cuda(op), cuda(rv)), exp):
            assert np.array_equal(g.cpu().numpy(), e)
        h.check_orders()
    # an order that is none, in one sample: the others come out as before, the call is reported
    if R > 1:
        chan = (np.arange(R) % 3).astype(np.int32)
        clean = tt.simulate_channels(h, 3, chan, cuda(orders), cuda(op), cuda(rv))[0].cpu().numpy()
        alone = tt.simulate(h, cuda(orders), cuda(op), cuda(rv))[0].cpu().numpy()
        for twice in (True, False):
            bad = orders.copy()
            bad[7, R - 1] = bad[7, 0] if twice else R
            got = tt.simulate_channels(h, 3, chan, cuda(bad), cuda(op), cuda(rv))[0].cpu().numpy()
            assert np.array_equal(np.delete(got, 7), np.delete(clean, 7))
            with pytest.raises(tt.TicTacError):
                h.check_orders()
            got = tt.simulate(h, cuda(bad), cuda(op), cuda(rv))[0].cpu().numpy()
            assert np.array_equal(np.delete(got, 7), np.delete(alone, 7))
            with pytest.raises(tt.TicTacError):
                h.check_orders()
            tt.simulate(h, cuda(bad[7]), cuda(op), cuda(rv))
            with pytest.raises(tt.TicTacError):
                h.check_orders()


# more classes than the registers of a lane hold, about as many recvs as are tried first, rows with few and with all recvs
RELEASES = {f"layered{r}": (lambda r=r: layered(45, 30, r, (2, 9))) for r in (4, 31, 32, 33, 63, 65, 192, 300, 511, 512)}
RELEASES["wide"] = lambda: layered(4, 300, 260, (3, 12))
RELEASES["chain512"] = lambda: chain(512, 40)


@pytest.mark.parametrize("name", list(RELEASES))
def test_release_positions(tt, name):
    d = RELEASES[name]()
    R, B = d.n_recv, 29
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(*args)
    rng = np.random.default_rng(8)
    orders = np.stack([rng.permutation(R) for _ in range(B)]).astype(np.int32)
    op = rng.integers(0, 50, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(0, 50, size=(B, R)).astype(np.float64) * wl.QUANTUM
    print(f"[releases] {name}: classes={h.n_classes} R={R}", flush=True)
    for o in (orders, orders[0]):
        exp = oracle.simulate(*args, o, op, rv)
        for g, e in zip(tt.simulate(h, cuda(o), cuda(op), cuda(rv)), exp):
            assert np.array_equal(g.cpu().numpy(), e)
        for g, e in zip(tt.simulate(h, cuda(o), cuda(op).float(), cuda(rv).float()), exp):     # (float32 holds the values)
            assert np.array_equal(g.cpu().numpy(), e)
    h.check_orders()
    clean = tt.simulate(h, cuda(orders), cuda(op), cuda(rv))[0].cpu().numpy()
    for wrong in (orders[7, 0], R, -1):
        bad = orders.copy()
        bad[7, R - 1] = wrong
        got = tt.simulate(h, cuda(bad), cuda(op), cuda(rv))[0].cpu().numpy()
        assert np.array_equal(np.delete(got, 7), np.delete(clean, 7))
        with pytest.raises(tt.TicTacError):
            h.check_orders()
        tt.simulate(h, cuda(bad[7]), cuda(op), cuda(rv))
        with pytest.raises(tt.TicTacError):
            h.check_orders()


# class slots per lane (one register kernel for each, two slots apart above eight), words of the rows, waves that fit
SLOTS = {
    "chain385": lambda: chain(385), "chain1000": lambda: chain(1000, 1),
    "few_classes": lambda: layered(3, 12, 700, (2, 5)),
    "k4": lambda: layered(20, 10, 500), "k6": lambda: layered(25, 15, 640), "k6_1024": lambda: layered(25, 15, 1024),
    "k8": lambda: layered(40, 20, 203), "k10": lambda: layered(50, 20, 203), "k10_short": lambda: layered(40, 20, 61), "k9_wide": lambda: layered(30, 20, 400),
    "k13": lambda: layered(61, 23, 203), "k13_wide": lambda: layered(50, 20, 500), "k15": lambda: layered(58, 23, 380),
    "k16": lambda: layered(65, 24, 330),
}


@pytest.mark.parametrize("name", list(SLOTS))
def test_tac_in_registers(tt, name):
    d = SLOTS[name]()
    R, B = d.n_recv, 37
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(*args)
    assert h.n_classes <= 1024, h.n_classes
    dep = oracle.find_dependencies(*args)
    rng = np.random.default_rng(9)
    rows = [0, 17, 36]

    def ints(lo, hi, n):
        return rng.integers(lo, hi, size=(B, n)).astype(np.float64) * wl.QUANTUM

    zero = ints(1, 1 << 20, R)
    zero[::5, 0] = 0.0                      # (these go to the general kernel, between the others)
    for what, op, rv in (("distinct", ints(1, 1 << 20, d.n_compute), ints(1, 1 << 20, R)),
                         ("ties", ints(0, 3, d.n_compute), ints(1, 4, R)),
                         ("zeros", ints(0, 1 << 20, d.n_compute), zero)):
        print(f"[registers] {name} {what}: classes={h.n_classes} R={R}", flush=True)
        got = tt.tac_simulate(h, cuda(op), cuda(rv), want_rank=True)
        eo, er = oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[:2]
        assert np.array_equal(got[0].cpu().numpy()[rows], eo), what
        assert np.array_equal(got[1].cpu().numpy()[rows], er), what
        exp = oracle.simulate(*args, eo, op[rows], rv[rows])
        for g, e in zip(got[4:9], exp):     # (integers times a power of two: every sum is exact)
            assert np.array_equal(g.cpu().numpy()[rows], e), what


# ---- several samples per wave, several waves per workgroup: more samples than the chip holds at a time ----
MANY = 9001                                 # sixteen waves on each of 256 compute units, twice over, and a few more


def copies(a, n=MANY):
    """n rows: those of ``a`` over and over (an odd number of rows, so that the copies of one fall to different waves)."""
    return cuda(a)[torch.arange(n, device="cuda") % len(a)].contiguous()


def same_in_every_copy(got, first):
    for g, f in zip(got, first):
        f = f if torch.is_tensor(f) else cuda(f)
        assert torch.equal(g, f[torch.arange(len(g), device="cuda") % len(f)])


@pytest.mark.parametrize("name", ["k4", "k8", "k10", "k13", "k13_wide", "k16", "chain1000"])
def test_tac_in_registers_many_samples(tt, name):
    d = SLOTS[name]()
    R, B = d.n_recv, 37
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(*args)
    dep = oracle.find_dependencies(*args)
    rng = np.random.default_rng(10)
    op = rng.integers(0, 1 << 20, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(1, 1 << 20, size=(B, R)).astype(np.float64) * wl.QUANTUM
    op[::3], rv[::3] = np.floor(op[::3] / wl.QUANTUM % 3) * wl.QUANTUM, np.floor(rv[::3] / wl.QUANTUM % 3 + 1) * wl.QUANTUM      # (ties)
    rv[4::9, 0] = 0.0                       # (the general kernel's, between the others)
    first = tt.tac_simulate(h, cuda(op), cuda(rv), want_rank=True)
    rows = [0, 4, 5, 36]
    eo = oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[0]
    assert np.array_equal(first[0].cpu().numpy()[rows], eo)
    for n in (2048, 2049, MANY):            # (eight samples per compute unit, the most that the kernel with more registers takes)
        print(f"[registers] {name}: classes={h.n_classes} R={R} B={n}", flush=True)
        many = tt.tac_simulate(h, copies(op, n), copies(rv, n), want_rank=True)
        same_in_every_copy([many[k] for k in (0, 1, 4, 5, 6, 7, 8)], [first[k] for k in (0, 1, 4, 5, 6, 7, 8)])


@pytest.mark.parametrize("name", ["layered300", "layered63", "wide", "two_words"])
def test_release_positions_many_samples(tt, name):
    # (the last: small batches are a workgroup's per sample, these a wave's)
    d = layered(40, 130, 100) if name == "two_words" else RELEASES[name]()
    R, B = d.n_recv, 29
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(*args)
    assert name != "two_words" or h.n_classes > 2048
    rng = np.random.default_rng(11)
    orders = np.stack([rng.permutation(R) for _ in range(B)]).astype(np.int32)
    op = rng.integers(0, 50, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(0, 50, size=(B, R)).astype(np.float64) * wl.QUANTUM
    print(f"[releases] {name}: classes={h.n_classes} R={R} B={MANY}", flush=True)
    for n in (B, 256, 257, MANY):
        same_in_every_copy(tt.simulate(h, copies(orders, n), copies(op, n), copies(rv, n)), oracle.simulate(*args, orders, op, rv))
    same_in_every_copy(tt.simulate(h, cuda(orders[0]), copies(op), copies(rv)), oracle.simulate(*args, orders[0], op, rv))
    h.check_orders()


@pytest.mark.parametrize("name", ["many_classes28", "many_classes300", "chain193"])
def test_consecutive_positions_many_samples(tt, name):
    d = POSITIONS[name]()
    R, B = d.n_recv, 23
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    h = tt.build_deps(*args)
    rng = np.random.default_rng(12)
    orders = np.stack([rng.permutation(R) for _ in range(B)]).astype(np.int32)
    op = rng.integers(0, 50, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
    rv = rng.integers(0, 50, size=(B, R)).astype(np.float64) * wl.QUANTUM
    chan = rng.integers(0, 3, size=R).astype(np.int32)
    print(f"[positions] {name}: classes={h.n_classes} R={R} B={MANY}", flush=True)
    same_in_every_copy(tt.simulate_channels(h, 3, chan, copies(orders), copies(op), copies(rv)),
                       oracle.simulate_channels(*args, 3, chan, orders, op, rv))
    moves = rng.integers(0, R, size=(64, 2)).astype(np.int32)
    same_in_every_copy(tt.order_search(h, copies(orders), cuda(moves), copies(op), copies(rv)),
                       oracle.order_search(*args, orders, moves, op, rv))
    h.check_orders()
