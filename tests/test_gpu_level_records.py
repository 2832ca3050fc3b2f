"""GPU parity of the dependency sets of graphs whose level-major records a kernel makes: no lists of inputs, lists that fit
LDS, and more than fit it; rows formed on the host and by the kernels; one graph and several by one launch."""

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


def layered(levels, width, recvs, far, wide, seed=1):
    """Three inputs per op from the two levels before; a share ``far`` of the ops has one from any level before, a share
    ``wide`` has six inputs and three recvs."""
    rng = np.random.default_rng(seed)
    row, col = [0] * (recvs + 1), []
    for l in range(levels):
        for j in range(width):
            ins = set()
            if l:
                ins.update((recvs + rng.integers(max(0, l - 2) * width, l * width, size=3)).tolist())
                if rng.random() < far:
                    ins.add(recvs + int(rng.integers(0, l * width)))
            if rng.random() < wide:
                ins.update(rng.integers(0, recvs, size=3).tolist())
                if l:
                    ins.update((recvs + rng.integers(max(0, l - 2) * width, l * width, size=3)).tolist())
            elif rng.random() < 0.1 or not l:
                ins.add(int(rng.integers(0, recvs)))
            col += sorted(ins)
            row.append(len(col))
    n = recvs + levels * width
    return wl.Dag("records", n, np.array(row, np.int32), np.array(col, np.int32), np.arange(recvs, dtype=np.int32),
                  np.ones(n - recvs), np.ones(recvs))


@pytest.mark.parametrize("far,wide", [(0.0, 0.0), (0.01, 0.005), (0.6, 0.1)])
@pytest.mark.parametrize("levels,width,recvs", [(120, 70, 100), (65, 33, 130), (300, 100, 1300)])
def test_level_records(tt, levels, width, recvs, far, wide):
    d = layered(levels, width, recvs, far, wide)
    dep = oracle.find_dependencies(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    hs = [tt.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids) for _ in range(2)]
    print(f"[records] {levels}x{width} {recvs} far={far} wide={wide}: W={dep.shape[1]}", flush=True)
    for h in hs:
        assert np.array_equal(h.deps().cpu().numpy().view(np.uint64), dep)
        h.deps_view().zero_()
        h.recompute_deps()
        assert np.array_equal(h.deps().cpu().numpy().view(np.uint64), dep)
        h.deps_view().zero_()
    tt.recompute_deps_batch(hs)
    for h in hs:
        assert np.array_equal(h.deps().cpu().numpy().view(np.uint64), dep)
