"""Byte knobs at the interface's largest number of knobs (d = 32), where the matrix-core kernel has no knob slot to spare
for the centroid norms: sizes around its tiles, waves and limits, the whole byte range, against the oracle and
the all-double path."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import check_pipeline, check_sweep, run_both

pytestmark = pytest.mark.gpu


def _check(wl, want_trace=False, path=0):
    import torch
    dw, g, c = run_both(wl, threshold=1.05, want_trace=want_trace)
    assert binding.cham_sweep_path(dw.ld, dw.d, wl.task_off, wl.ks) == path
    check_sweep(wl, g["sweep"], c, dw.ld)
    check_pipeline(wl, g, c)
    ex = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, flags=binding.F_FORCE_EXACT)
    torch.cuda.synchronize()
    for key in ("status", "counts", "centroids", "labels"):
        assert torch.equal(ex[key], g["sweep"][key]), key


@pytest.mark.parametrize("n,ks", [(1, (1,)), (31, (1, 5)), (129, (2, 33)), (1024, (7, 32, 64)), (1025, (8, 31, 63)), (2048, (2, 16, 64)),
                                  (2049, (2, 16, 32)), (4096, (1, 9, 24, 32))])
def test_sizes(n, ks):
    wl = workloads.random_task(n + len(ks), n, 32, card_hi=40, n_blobs=9, sigma=1.2, invalid_frac=0.05, ks=ks, n_iter=20, n_visited=50,
                               n_tasks=2, ragged=n % 2 == 1)
    _check(wl)


def test_above_the_limits():
    wl = workloads.random_task(5, 2049, 32, card_hi=40, n_blobs=9, ks=(4, 33), n_iter=6)
    _check(wl, path=2)


def test_trace_and_duplicates():
    wl = workloads.random_task(6, 1500, 32, card_lo=1, card_hi=3, n_blobs=3, sigma=0.4, ks=(1, 2, 3, 40, 64), n_iter=12, n_tasks=2)
    _check(wl, want_trace=True)


@pytest.mark.parametrize("n,k", [(900, 64), (2000, 64), (4000, 32)])
def test_whole_byte_range(n, k):
    rng = np.random.default_rng(n)
    wl = workloads.random_task(n, n, 32, card_lo=256, card_hi=256, n_blobs=8, sigma=30.0, ks=(3, k), n_iter=15)
    wl.rows[:: 3, ::2] = rng.choice([0, 255], size=wl.rows[:: 3, ::2].shape)      # far from the centring offsets
    wl.rows[1::7] = wl.rows[2]                                                       # and many duplicates
    _check(wl)
