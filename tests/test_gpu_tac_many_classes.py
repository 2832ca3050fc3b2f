"""GPU parity of TAC with more than 512 and up to 1 024 classes of compute ops (the wave-per-sample kernel with nine to
sixteen classes per lane): at the edges of its class slots, on times with and without ties, with batches that leave waves
without a sample, against the CPU oracle."""

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


def pairs_dag(n_classes, n_recv):
    """Ops that read one or two recvs each, no two the same set: n_classes classes over n_recv recvs."""
    b = wl._Builder()
    rs = [b.recv(1e5 * (1 + k % 7)) for k in range(n_recv)]
    sets = [(i,) for i in range(n_recv)] + [(i, j) for d in range(1, n_recv) for i in range(n_recv - d) for j in (i + d,)]
    for k, s in enumerate(sets[:n_classes]):
        b.op([rs[i] for i in s], 1e-3 * (1 + k % 5), "op")
    return b.finish("pairs", seed=3, batch=4)


def layered(levels, width, recvs):
    return wl.layered_dag(41, levels=levels, width=width, fan_in=(1, 3), back=3, n_recv=recvs, attach=(1, 3))


GRAPHS = {
    "pairs513": lambda: pairs_dag(513, 40),
    "pairs640": lambda: pairs_dag(640, 64),
    "pairs641": lambda: pairs_dag(641, 65),
    "pairs896": lambda: pairs_dag(896, 129),
    "pairs1023": lambda: pairs_dag(1023, 384),      # more pointers than lanes at the start
    "pairs1024": lambda: pairs_dag(1024, 100),
    "pairs1025": lambda: pairs_dag(1025, 100),      # one too many
    "layered651": lambda: layered(40, 23, 203),
    "layered904": lambda: layered(30, 40, 384),
    "layered1011": lambda: layered(34, 40, 380),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_tac_with_many_classes(tt, name):
    d = GRAPHS[name]()
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rng = np.random.default_rng(7)
    B = 37
    cases = [("distinct", rng.integers(1, 1 << 20, size=(B, d.n_compute)), rng.integers(1, 1 << 20, size=(B, d.n_recv))),
             ("ties", rng.integers(0, 3, size=(B, d.n_compute)), rng.integers(1, 4, size=(B, d.n_recv)))]
    for what, op, rv in cases:
        op, rv = op.astype(np.float64) * wl.QUANTUM, rv.astype(np.float64) * wl.QUANTUM
        print(f"[tac] {name} {what}: classes={h.n_classes} R={d.n_recv}", flush=True)
        order, rank = (x.cpu().numpy() for x in tt.tac_priority(h, torch.from_numpy(op).cuda(), torch.from_numpy(rv).cuda())[:2])
        rows = list(range(0, B, 3))
        eo, er = oracle_tac_rows(dep, d.recv_ids, op[rows], rv[rows])[:2]
        assert np.array_equal(order[rows], eo), what
        assert np.array_equal(rank[rows], er), what
    h.close()


@pytest.mark.parametrize("levels,width,recvs,low,high", [(20, 20, 200, 321, 384), (24, 20, 300, 385, 448), (50, 18, 203, 513, 640), (45, 22, 203, 641, 768), (61, 23, 203, 769, 896), (60, 28, 203, 897, 1024)])
def test_two_sets_of_waves(tt, levels, width, recvs, low, high):
    """Batches whose samples take two sets of sixteen waves per compute unit (of twelve, above 512 classes): dealt to the sets evenly, they give
    every sample what batches of one set give."""
    d = wl.layered_dag(41, levels=levels, width=width, fan_in=(1, 4), back=3, n_recv=recvs, attach=(1, 8))
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    print(f"[tac] two sets: {levels} x {width}, {recvs}: classes={h.n_classes}", flush=True)
    assert low <= h.n_classes <= high, h.n_classes
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator(device="cuda").manual_seed(levels)
    for B in (16 * cu + 1, 20 * cu - 117, 24 * cu):
        op = torch.randint(1, 1 << 20, (B, d.n_compute), device="cuda", generator=gen).double() * wl.QUANTUM
        rv = torch.randint(1, 1 << 20, (B, d.n_recv), device="cuda", generator=gen).double() * wl.QUANTUM
        got = tt.tac_simulate(h, op, rv, want_rank=True)
        for lo in range(0, B, 8 * cu):
            part = tt.tac_simulate(h, op[lo:lo + 8 * cu].contiguous(), rv[lo:lo + 8 * cu].contiguous(), want_rank=True)
            for k in (0, 1, 4, 5, 6, 7, 8):
                assert torch.equal(got[k][lo:lo + 8 * cu], part[k]), (B, lo, k)
    h.close()


def test_one_and_two_words_per_lane(tt):
    """The bit-sliced kernel on a graph whose classes take two words per lane for a batch of more samples than compute
    units (two workgroups share one) and one word for a smaller batch: the same results for every sample."""
    d = wl.stress_dag(levels=220, width=200, n_recv=3000, seed=9, batch=8)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    assert 28672 < h.n_classes <= 57344, h.n_classes
    B = 300
    op, rv = (torch.from_numpy(x).cuda() for x in wl.timing_samples(d, 0, B))
    print(f"[tac] words per lane: classes={h.n_classes} R={d.n_recv}", flush=True)
    got = tt.tac_simulate(h, op, rv, want_rank=True)
    for lo in range(0, B, 150):
        part = tt.tac_simulate(h, op[lo:lo + 150].contiguous(), rv[lo:lo + 150].contiguous(), want_rank=True)
        for k in (0, 1, 4, 5, 6, 7, 8):
            assert torch.equal(got[k][lo:lo + 150], part[k]), (lo, k)
    h.close()
