"""More tasks than one launch of the packing kernel has workgroups for: tiny ones beside one whose rows are fetched in every pass."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding

pytestmark = pytest.mark.gpu


def test_a_million_tiny_tasks_beside_a_large_one():
    import torch
    T, d, big = 1_048_700, 3, 4096                # sixteen workgroups a task: 2^32 threads and more
    sizes = np.full(T, 2, dtype=np.int64)
    sizes[T - 3] = big
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    rng = np.random.default_rng(0)
    rows = rng.integers(0, 40, size=(n, d), dtype=np.uint8)
    X, ld = binding.to_soa(rows)
    assert binding.cham_sweep_kernel(ld, d, off, (1, 2)) == "resident_mfma_kernel"
    out = binding.cham_kmeans_sweep(X, ld, d, off, (1, 2), 2, want_labels=True)
    torch.cuda.synchronize()
    ref = oracle.sweep(rows, off, (1, 2), 2, want_labels=True)
    np.testing.assert_array_equal(out["status"].cpu().numpy(), ref["status"])
    np.testing.assert_array_equal(out["counts"].cpu().numpy(), ref["counts"])
    np.testing.assert_array_equal(out["centroids"].cpu().numpy(), ref["centroids"])
    np.testing.assert_array_equal(out["labels"].cpu().numpy()[:, :n], ref["labels"])
    np.testing.assert_allclose(out["inertia"].cpu().numpy(), ref["inertia"], rtol=1e-11, atol=0)
