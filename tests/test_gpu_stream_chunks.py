"""The streaming sweep's row chunks and settled units: sizes around the chunk lengths (512 to 4096 rows), launches with
fewer and with more workgroups than places on the chip, iterations that settle long before the last pass."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import check_sweep

pytestmark = pytest.mark.gpu


def _sweep(wl, want_trace=False, init=None):
    import torch
    dw = binding.DeviceWorkload(wl)
    kw = {} if init is None else dict(init_centroids=torch.from_numpy(init).to(dw.X.device))
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=want_trace,
                                    flags=binding.F_STREAMING, **kw)
    torch.cuda.synchronize()
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, init=init, want_labels=True, want_trace=want_trace)
    check_sweep(wl, out, ref, dw.ld)
    return dw, out


@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 1024, 1025, 2049, 4095, 4097, 8193])
@pytest.mark.parametrize("d,ks", [(16, (1, 3, 40)), (17, (2, 65, 130)), (31, (1, 33, 256))])
def test_chunk_edges(n, d, ks):
    wl = workloads.random_task(n * 40 + d, n, d, card_hi=20, n_blobs=6, sigma=0.7, ks=ks, n_iter=25, n_tasks=2, ragged=n % 2 == 1)
    _sweep(wl)


@pytest.mark.parametrize("n_iter", [0, 1, 2, 40])
@pytest.mark.parametrize("want_trace", [False, True])
def test_settled_units(n_iter, want_trace):
    # k = 1 settles in its second pass, the other units after some; a traced sweep runs every pass
    wl = workloads.random_task(77, 3000, 12, card_hi=12, n_blobs=4, sigma=0.5, ks=(1, 2, 4, 70), n_iter=n_iter, n_tasks=3, ragged=True)
    _sweep(wl, want_trace)


def test_more_units_than_places():
    # 40 tasks x 16 values of k > 512 workgroups of 4096 rows
    wl = workloads.random_task(78, 700, 9, card_hi=16, n_blobs=5, sigma=0.8, ks=tuple(range(1, 17)), n_iter=12, n_tasks=40, ragged=True)
    _sweep(wl)


def test_starts_at_a_fixed_point():
    # the centroids of a settled run as the start: the second pass moves nothing
    wl = workloads.random_task(79, 2600, 10, card_hi=14, n_blobs=5, sigma=0.6, ks=(3, 66), n_iter=60, n_tasks=2)
    _, out = _sweep(wl)
    wl.n_iter = 9
    _sweep(wl, init=out["centroids"].cpu().numpy())


def test_chunked_sweep_equals_the_whole():
    import torch
    wl = workloads.random_task(80, 5000, 14, card_hi=18, n_blobs=6, sigma=0.8, ks=(2, 4, 8, 16, 32), n_iter=15, n_tasks=5, ragged=True)
    dw, whole = _sweep(wl)
    part = binding.cham_kmeans_sweep_knee(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, threshold=0.0, chunk=2, want_labels=True,
                                          flags=binding.F_STREAMING)
    torch.cuda.synchronize()
    for key in ("status", "counts", "centroids", "labels", "inertia"):
        assert torch.equal(part[key], whole[key]), key


@pytest.mark.parametrize("n_iter", [0, 1, 2, 3, 25])
def test_passes_of_settled_units(n_iter):
    # as the resident kernel: up to and including the pass that moves no row
    wl = workloads.random_task(81, 3000, 12, card_hi=12, n_blobs=4, sigma=0.5, ks=(1, 2, 4, 20, 64), n_iter=n_iter, n_tasks=3, ragged=True)
    dw, out = _sweep(wl)
    ran = binding.cham_sweep_passes(out["workspace"], dw.ld, dw.d, wl.task_off, wl.ks, flags=binding.F_STREAMING).cpu().numpy()
    res = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, n_iter)
    stops = binding.cham_sweep_passes(res["workspace"], dw.ld, dw.d, wl.task_off, wl.ks).cpu().numpy()
    np.testing.assert_array_equal(ran, stops)
    if n_iter == 25:
        assert ran.min() < n_iter + 1
    _, traced = _sweep(wl, want_trace=True)
    ran = binding.cham_sweep_passes(traced["workspace"], dw.ld, dw.d, wl.task_off, wl.ks, flags=binding.F_STREAMING).cpu().numpy()
    assert (ran == n_iter + 1).all()
