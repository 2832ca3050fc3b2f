"""GPU parity of the straight form of the iteration with sends at the sizes where its ways to read the times change: recvs and
columns with sends that just fit the space of the tiles or just do not, one recv, one send, sends in the first and the last
columns, batches around a group of 64 samples."""

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


def chain_with_sends(recvs, extra, sends, first):
    """A chain of ``recvs`` ops with a recv each and ``extra`` ops without; a send behind the first (``first``) or the last
    ``sends`` of them, at the end of the columns."""
    n_chain = recvs + extra
    row, col = [0] * (recvs + 1), []
    for k in range(n_chain):
        col += ([recvs + k - 1] if k else []) + ([k] if k < recvs else [])
        row.append(len(col))
    behind = range(sends) if first else range(n_chain - sends, n_chain)
    for k in behind:
        col.append(recvs + k)
        row.append(len(col))
    n = recvs + n_chain + sends
    d = wl.Dag("straight", n, np.array(row, np.int32), np.array(col, np.int32), np.arange(recvs, dtype=np.int32),
               np.ones(n - recvs), np.ones(recvs))
    return d, np.arange(recvs + n_chain, n, dtype=np.int32)


@pytest.mark.parametrize("recvs,extra,sends,first", [(1, 1, 1, True), (2, 61, 1, False), (64, 0, 63, True), (65, 3, 66, False),
                                                     (190, 1, 191, False), (191, 2, 192, True), (192, 70, 190, False), (300, 0, 300, True),
                                                     # batches of sixteen, eight and four loads; sixteen recvs or sends and one more
                                                     (3, 1, 4, True), (4, 13, 16, False), (16, 0, 16, True), (17, 0, 17, False), (16, 3, 17, True),
                                                     (17, 9, 16, False), (33, 0, 33, True), (36, 4, 37, False), (63, 1, 64, True), (64, 0, 64, False),
                                                     (64, 2, 65, True), (65, 0, 64, False), (96, 8, 100, True), (100, 8, 97, False)])
def test_straight_form(tt, recvs, extra, sends, first):
    d, ids = chain_with_sends(recvs, extra, sends, first)
    h = tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    args = (d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    rng = np.random.default_rng([recvs, sends])
    for B in (1, 63, 65, 130):
        op = rng.integers(1, 3000, size=(B, d.n_compute)).astype(np.float64) * wl.QUANTUM
        rv = rng.integers(1, 2000, size=(B, recvs)).astype(np.float64) * wl.QUANTUM
        each = np.stack([rng.permutation(recvs) for _ in range(B)]).astype(np.int32)
        print(f"[straight] R={recvs} N={d.n_compute} sends={sends} B={B}", flush=True)
        for order in (np.arange(recvs, dtype=np.int32), each):
            got = tt.simulate_sends(h, ids, *(torch.from_numpy(x).cuda() for x in (order, op, rv)))
            exp = oracle.simulate_sends(*args, ids, order, op, rv)
            for k, name in enumerate("m E U L S".split()):
                a = got[k].cpu().numpy()
                if name in "mUL":
                    assert np.array_equal(a, exp[k]), (B, name)         # (multiples of a quantum: sums are exact)
                else:
                    np.testing.assert_allclose(a, exp[k], rtol=1e-12, atol=1e-12)
    h.check_orders()
    h.close()
