"""The resident matrix-core sweep's splits of a task over waves: sizes around every number of tiles per wave, few and many
units, 16-, 32-, 48- and 64-wide rows, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import check_sweep

pytestmark = pytest.mark.gpu


def _sweep(wl, flags=0, want_trace=False, sfx=None):
    import torch
    dw = binding.DeviceWorkload(wl)
    kw = {} if sfx is None else dict(_sfx=sfx)
    assert (binding.cham_sweep_path_u16 if sfx else binding.cham_sweep_path)(dw.ld, dw.d, wl.task_off, wl.ks, flags=flags) == 0
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=want_trace, flags=flags, **kw)
    torch.cuda.synchronize()
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=want_trace)
    check_sweep(wl, out, ref, dw.ld)


@pytest.mark.parametrize("n", [1, 64, 65, 511, 512, 513, 1023, 1025, 2047, 2049])
@pytest.mark.parametrize("d,ks", [(3, (1, 2, 9)), (15, (2, 31, 33, 64)), (16, (3, 17, 32)), (31, (5, 40, 64))])
def test_sizes_of_byte_knobs(n, d, ks):
    wl = workloads.random_task(7 * n + d, n, d, card_hi=24, n_blobs=7, sigma=1.0, ks=ks, n_iter=18, n_tasks=3, ragged=n % 2 == 1)
    _sweep(wl, want_trace=n == 513)


@pytest.mark.parametrize("n,d,tasks,ks", [(500, 9, 40, range(2, 12)), (1024, 28, 30, range(2, 20)), (2000, 24, 20, range(10, 40))])
def test_more_units_than_places(n, d, tasks, ks):
    # (500: more than 256 units; 2000: more than 512 units with more than 32 centroids)
    wl = workloads.random_task(n, n, d, card_hi=24, n_blobs=7, sigma=1.0, ks=tuple(ks), n_iter=6, n_tasks=tasks, ragged=True)
    _sweep(wl)


@pytest.mark.parametrize("n", [1, 129, 1024, 1025, 2048])
@pytest.mark.parametrize("d", [33, 44, 47, 48, 63])
def test_sizes_of_two_byte_knobs(n, d):
    wl = workloads.wide_space(n + d, n_tasks=2, n=n, d=d, ks=(1, 7, 32), n_iter=14, card_wide=(64, 2048), ragged=n % 2 == 1)
    wl.rows[: max(1, len(wl.rows) // 3)] = wl.rows[0]          # a cluster of duplicates
    _sweep(wl, flags=binding.F_VALUES_BELOW_2048, sfx="_u16")
