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
    d = SMALL[name]() if name in SMALL else wl.preset(name)
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
