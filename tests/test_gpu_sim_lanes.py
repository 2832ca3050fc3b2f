"""GPU parity of the one-lane-per-sample simulation of small graphs: one order for all samples at any batch, an order per
sample on large batches, against the wave-per-sample kernel (smaller batches) on every sample and the CPU oracle on some."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle
from paper_1803_03288_amd import workloads as wl


@pytest.fixture(scope="module")
def tt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1803_03288_amd import binding
    binding.lib()
    return binding


GRAPHS = {
    "toy": wl.toy_dag,
    "single": lambda: wl.chain_dag(1),
    "case2": wl.case2_dag,
    "chain63": lambda: wl.chain_dag(63),
    "chain128": lambda: wl.chain_dag(128),          # 256 rows: the largest (float64 does not fit, float32 does)
    "jobs": lambda: wl.independent_jobs_dag(9),
    "funnel": lambda: wl.funnel_dag(70, 90),        # two words per row, one class
    "tiny": wl.tiny_dag,
    "vgg16": wl.vgg16_dag,
    "layered": lambda: wl.layered_dag(31, levels=8, width=7, fan_in=(1, 3), back=2, n_recv=50, attach=(1, 3)),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_simulate_lanes(tt, name):
    d = GRAPHS[name]()
    rng = np.random.default_rng(len(name))
    B = 24 * 1024 + 64 + 29
    op = wl.quantise(1e-3 * np.exp(0.5 * rng.standard_normal((B, d.n_compute))))
    rv = wl.quantise(1e-3 * np.exp(0.5 * rng.standard_normal((B, d.n_recv))))
    order = np.argsort(rng.random((B, d.n_recv)), axis=1).astype(np.int32)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    gop, grv, gord = (torch.from_numpy(x).cuda() for x in (op, rv, order))
    print(f"[lanes] {name}: N={d.n_compute} R={d.n_recv} classes={h.n_classes}", flush=True)
    rows = np.linspace(0, B - 1, 50).astype(int)
    for f32 in (False, True):
        o, r = (gop.float(), grv.float()) if f32 else (gop, grv)
        got = tt.simulate(h, gord, o, r)
        for lo in range(0, B, 8192):
            part = tt.simulate(h, gord[lo:lo + 8192].contiguous(), o[lo:lo + 8192].contiguous(), r[lo:lo + 8192].contiguous())
            for k in range(5):
                assert torch.equal(got[k][lo:lo + 8192], part[k]), (name, f32, k, lo)
        exp = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, order[rows], o[rows].double().cpu().numpy(),
                              r[rows].double().cpu().numpy())
        for k in range(5):
            np.testing.assert_allclose(got[k][rows].cpu().numpy(), exp[k], rtol=1e-12, atol=0)
        # the order of sample 0 for all: in one row, and repeated
        one = gord[0].contiguous()
        shared, each = tt.simulate(h, one, o, r), tt.simulate(h, one.expand(B, -1).contiguous(), o, r)
        few = tt.simulate(h, one, o[:3].contiguous(), r[:3].contiguous())
        for k in range(5):
            assert torch.equal(shared[k], each[k]) and torch.equal(shared[k][:3], few[k])
    h.check_orders()


def chain_of(ops, recvs):
    """A chain of ops, the first ones with a recv each."""
    b = wl._Builder()
    rs, x = [b.recv(1e5) for _ in range(recvs)], []
    for k in range(ops):
        x = [b.op(x + (rs[k:k + 1] if k < ops - 1 else rs[k:]), 1e-3, "op")]
    return b.finish("chain_of", seed=3, batch=4)


# One order for all, rows of the next samples requested ahead: pieces of 32 columns (float64) or 64 (float32), one or two of op_time's rows
# and one of recv_time's; rows as long as a request, a column more, and so long that nothing is requested ahead.
@pytest.mark.parametrize("ops,recvs", [(2, 2), (3, 2), (4, 4), (5, 3), (31, 8), (32, 32), (33, 32), (40, 33), (63, 17), (64, 31), (64, 64), (65, 32),
                                       (90, 64), (127, 63), (128, 64), (128, 65), (129, 64)])
def test_more_samples_than_are_under_way(tt, ops, recvs):
    """Every wave takes several groups of 64 samples, the last one not whole."""
    d = chain_of(ops, recvs)
    B, part = 64 * 256 * 16 + 64 * 5 + 29, 16384                # (at most sixteen such waves share a compute unit)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    gen = torch.Generator(device="cuda").manual_seed(ops)
    op = torch.randint(0, 1 << 14, (B, ops), device="cuda", generator=gen) * 2.0 ** -20
    rv = torch.randint(0, 1 << 14, (B, recvs), device="cuda", generator=gen) * 2.0 ** -20
    order = torch.randperm(recvs, device="cuda", generator=gen).to(torch.int32)
    rows = [0, 63, 64, part, B // 2, B - 30, B - 1]
    for dtype in (torch.float64, torch.float32):
        print(f"[lanes] {ops} ops, {recvs} recvs, {dtype}, {B} samples", flush=True)
        o, r = op.to(dtype), rv.to(dtype)
        got = tt.simulate(h, order, o, r)
        for lo in range(0, B, part):
            for x, y in zip(got, tt.simulate(h, order, o[lo:lo + part].contiguous(), r[lo:lo + part].contiguous())):
                assert torch.equal(x[lo:lo + part], y), lo
        exp = oracle.simulate(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids, order.cpu().numpy()[None].repeat(len(rows), 0),
                              o[rows].double().cpu().numpy(), r[rows].double().cpu().numpy())
        for x, y in zip(got, exp):
            np.testing.assert_allclose(x[rows].cpu().numpy(), y, rtol=1e-12, atol=0)
    h.check_orders()


@pytest.mark.parametrize("value", [-1, 7, 1 << 20, "twice"])
def test_bad_orders_in_the_lane_kernels(tt, value):
    """An entry out of range or a recv named twice, in one sample of a large batch and in a shared order: reported, and
    the other samples are unaffected."""
    d = GRAPHS["layered"]()
    B = 24 * 1024 + 5
    rng = np.random.default_rng(3)
    op = torch.from_numpy(wl.quantise(1e-3 * rng.random((B, d.n_compute)))).cuda()
    rv = torch.from_numpy(wl.quantise(1e-3 * rng.random((B, d.n_recv)))).cuda()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    good = torch.arange(d.n_recv, dtype=torch.int32, device="cuda")
    ref = tt.simulate(h, good, op, rv)
    h.check_orders()
    bad_row = good.clone()
    bad_row[4] = int(good[9]) if value == "twice" else (value if value != 7 else d.n_recv)
    orders = good.expand(B, -1).clone()
    orders[77] = bad_row
    got = tt.simulate(h, orders, op, rv)
    with pytest.raises(tt.TicTacError):
        h.check_orders()
    keep = torch.arange(B, device="cuda") != 77
    for k in range(5):
        assert torch.equal(got[k][keep], ref[k][keep])
    tt.simulate(h, bad_row, op, rv)
    with pytest.raises(tt.TicTacError):
        h.check_orders()
    h.check_orders()
