"""Where the binding's output tensors lie: aligned like allocations of their own, and large ones kept alone."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1803_03288_amd import binding, workloads as wl


def check(tensors, size):
    for t in tensors:
        assert t.shape == (size,) and t.is_contiguous()
        assert (t.storage_offset() * t.element_size()) % 512 == 0
        kept = t.untyped_storage().nbytes()
        assert kept == size * t.element_size() or kept <= 5 * 8192
    spans = sorted((t.data_ptr(), t.data_ptr() + size * t.element_size()) for t in tensors)
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))


@pytest.mark.parametrize("dtype", [torch.float64, torch.int32])
@pytest.mark.parametrize("size", [1, 63, 64, 65, 127, 1023, 1024, 1025, 2048, 2049, 5003])
def test_vectors(size, dtype):
    check(binding._vectors(5, size, dtype, "cpu"), size)


def test_no_vectors_of_no_size():
    assert [t.shape for t in binding._vectors(3, 0, torch.int32, "cpu")] == [(0,)] * 3


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1, 33, 1025, 4099])
def test_outputs_of_the_calls(B):
    d = wl.preset("tiny")
    h = binding.build_deps(d.n_ops, d.row_ptr, d.col_idx, d.recv_ids)
    op, rv = (torch.from_numpy(x).cuda() for x in wl.timing_samples(d, 0, B))
    prio, order, rank = binding.tic_priority(h)
    check((prio, order, rank), d.n_recv)
    check(binding.simulate(h, order, op, rv), B)
    check(binding.simulate_channels(h, 2, np.arange(d.n_recv) % 2, order, op, rv), B)
    check(binding.simulate_sends(h, [], order, op, rv), B)
    out = binding.tac_simulate(h, op, rv, want_rank=True)
    check(out[4:], B)
    for t in out[:2]:
        assert t.is_contiguous() and t.storage_offset() == 0 and t.untyped_storage().nbytes() == B * d.n_recv * 4
