"""Units that a sweep which stops at the knee skips: outputs of every length and alignment are zeroed, with all tasks
stopped, some or none, whatever the buffers held before."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import INERTIA_RTOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,flags", [(1, 5, 0), (61, 9, 0), (1500, 24, 0), (1500, 32, 0), (900, 12, binding.F_NO_MFMA), (900, 12, binding.F_STREAMING)])
@pytest.mark.parametrize("chunk,threshold", [(1, 1.05), (3, 2.5), (3, 1.05), (2, 0.0)])
def test_skipped_units(n, d, flags, chunk, threshold):
    import torch
    wl = workloads.random_task(n + d, n, d, card_hi=20, n_blobs=5, sigma=0.8, ks=(1, 2, 3, 5, 8, 13, 21), n_iter=8, n_tasks=5, ragged=True)
    dw = binding.DeviceWorkload(wl)
    T, n_k, ksum, dev = len(wl.task_off) - 1, len(wl.ks), sum(wl.ks), dw.X.device
    out = dict(centroids=torch.full((T, ksum, d), 7.0, dtype=torch.float64, device=dev), counts=torch.full((T, ksum), 7, dtype=torch.int32, device=dev),
               inertia=torch.full((T, n_k), 7.0, dtype=torch.float64, device=dev), status=torch.full((T, n_k), 7, dtype=torch.int32, device=dev),
               chosen=torch.full((T,), 7, dtype=torch.int32, device=dev), labels=torch.full((n_k, dw.ld), 7, dtype=torch.uint8, device=dev),
               trace=torch.full((T, n_k, wl.n_iter + 1), 7.0, dtype=torch.float64, device=dev))
    keys = list(out)
    binding.cham_kmeans_sweep_knee(dw.X, dw.ld, d, wl.task_off, wl.ks, wl.n_iter, threshold=threshold, chunk=chunk, flags=flags, out=out)
    torch.cuda.synchronize()
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=True)
    loop = oracle.sweep_until_knee(wl.rows, wl.task_off, wl.ks, wl.n_iter, threshold)
    g = {key: out[key].cpu().numpy() for key in keys}
    np.testing.assert_array_equal(g["chosen"], loop["chosen_idx"])
    koff = np.concatenate([[0], np.cumsum(wl.ks)])
    for t in range(T):
        rows = slice(wl.task_off[t], wl.task_off[t + 1])
        knee, usable = int(g["chosen"][t]), ref["status"][t] == 0
        # the knee was found by a test, not by running out of k's, when a usable k before it passes the threshold
        before = [i for i in range(max(knee, 0)) if usable[i]]
        found = bool(before) and threshold * ref["inertia"][t][knee] >= ref["inertia"][t][before[-1]]
        last_run = (knee // chunk + 1) * chunk if found else n_k
        for i in range(n_k):
            c = slice(koff[i], koff[i + 1])
            if i < last_run:
                assert g["status"][t, i] == ref["status"][t, i]
                np.testing.assert_array_equal(g["counts"][t, c], ref["counts"][t, c])
                np.testing.assert_array_equal(g["centroids"][t, c], ref["centroids"][t, c])
                np.testing.assert_array_equal(g["labels"][i, rows], ref["labels"][i, rows])
                # (the oracle's are zero where a unit has too few distinct rows)
                np.testing.assert_allclose(g["inertia"][t, i], ref["inertia"][t, i], rtol=INERTIA_RTOL, atol=0)
                np.testing.assert_allclose(g["trace"][t, i], ref["trace"][t, i], rtol=INERTIA_RTOL, atol=0)
            else:
                assert g["status"][t, i] == 3 and g["inertia"][t, i] == 0
                for key in ("counts", "centroids"):
                    assert not g[key][t, c].any()
                assert not g["trace"][t, i].any() and not g["labels"][i, rows].any()
    assert (g["labels"][:, wl.task_off[-1]:] == 7).all()
