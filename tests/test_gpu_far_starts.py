"""Sweeps whose centred centroids leave the range of the matrix-core screen's f16 operands: starting centroids far outside the
knobs' range (the interface sets none), and two-byte knobs spread over their whole promised range.  Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import check_sweep

pytestmark = pytest.mark.gpu


def _sweep(wl, init=None, flags=0, sfx="", path=0, want_trace=False):
    import torch
    dw = binding.DeviceWorkload(wl)
    assert binding.cham_sweep_path(dw.ld, dw.d, wl.task_off, wl.ks, flags=flags, _sfx=sfx) == path
    kw = {} if init is None else dict(init_centroids=torch.from_numpy(init).to(dw.X.device))
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=want_trace, flags=flags, _sfx=sfx, **kw)
    torch.cuda.synchronize()
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, init=init, want_labels=True, want_trace=want_trace)
    check_sweep(wl, out, ref, dw.ld)


def _starts(wl, rng, far, share):
    """Means of three rows of the task each; a share of the centroids, or of their knobs, moved out by about `far`."""
    T, ksum, d = wl.T, sum(wl.ks), wl.d
    init = np.empty((T, ksum, d))
    for t in range(T):
        rows = wl.task_rows(t).astype(np.float64)
        init[t] = rows[rng.integers(0, len(rows), size=(ksum, 3))].mean(axis=1)
    if far:
        moved = rng.random((T, ksum)) < share
        moved[:, ::5] = False                       # (some stay)
        away = far * rng.choice([-1.0, 1.0], size=(T, ksum, d)) * (0.5 + rng.random((T, ksum, d)))
        init[moved] += away[moved]
    return init


@pytest.mark.parametrize("far", [0.0, 700.0, 800.0, 5e3, 1e5, 1e9])
@pytest.mark.parametrize("d,n,ks", [(32, 900, (3, 8, 40)), (32, 2000, (5, 33)), (32, 4000, (2, 24)), (12, 500, (3, 9)), (24, 3000, (4, 48))])
def test_starts_outside_the_byte_range(d, n, ks, far):
    rng = np.random.default_rng(n + d)
    wl = workloads.random_task(n, n, d, card_hi=40, n_blobs=9, sigma=1.5, ks=ks, n_iter=6, n_tasks=2, ragged=True)
    _sweep(wl, init=_starts(wl, rng, far, 0.5))


@pytest.mark.parametrize("d,n,ks", [(32, 1500, (3, 8, 30)), (32, 1000, (5, 50)), (12, 500, (4, 9)), (24, 3000, (6, 48))])
def test_all_starts_about_the_largest_norm_of_the_screen(d, n, ks):
    # squared norms on both sides of 65504 * 256: rows have to choose among such starts
    rng = np.random.default_rng(n + d)
    wl = workloads.random_task(n, n, d, card_lo=200, card_hi=256, n_blobs=9, sigma=40.0, ks=ks, n_iter=4, n_tasks=3)
    shape = (wl.T, sum(ks), d)
    far = np.sqrt(65504 * 256 / d) * (1.0 + 0.01 * rng.standard_normal(shape[:2]))[:, :, None]
    _sweep(wl, init=128.0 + far * rng.choice([-1.0, 1.0], size=shape))


@pytest.mark.parametrize("d,n,ks", [(16, 1500, (3, 64, 100)), (24, 5000, (5, 70)), (9, 4100, (40,))])
@pytest.mark.parametrize("far", [32752.0, 1e6, 1e9])
def test_streaming_starts_beyond_half_precision(d, n, ks, far):
    # twice a start's distance per knob on both sides of 65504
    rng = np.random.default_rng(n + d)
    wl = workloads.random_task(n, n, d, card_lo=100, card_hi=256, n_blobs=9, sigma=30.0, ks=ks, n_iter=4, n_tasks=2)
    shape = (wl.T, sum(ks), d)
    _sweep(wl, init=128.0 + far * (1.0 + 0.01 * rng.standard_normal(shape)) * rng.choice([-1.0, 1.0], size=shape), flags=binding.F_STREAMING, path=1)
    _sweep(wl, init=_starts(wl, rng, far, 0.5), flags=binding.F_STREAMING, path=1)


@pytest.mark.parametrize("far", [0.0, 3e3, 1e5])
@pytest.mark.parametrize("d,n,ks", [(44, 1000, (3, 17)), (47, 2048, (5, 32)), (60, 700, (4, 9)), (20, 1500, (6, 40))])
def test_starts_outside_the_two_byte_range(d, n, ks, far):
    rng = np.random.default_rng(n + d)
    wl = workloads.wide_space(n + d, n_tasks=2, n=n, d=d, ks=ks, n_iter=6, card_wide=(64, 2048), ragged=True)
    _sweep(wl, init=_starts(wl, rng, far, 0.5), flags=binding.F_VALUES_BELOW_2048, sfx="_u16")


@pytest.mark.parametrize("d,n,ks", [(20, 1500, (1, 6, 40)), (47, 2000, (1, 2, 9, 32)), (63, 900, (1, 3, 20))])
def test_values_0_and_2047(d, n, ks):
    # corners of the promised range: squared norms up to d * 2047^2, above what the f16 bias holds
    rng = np.random.default_rng(d)
    wl = workloads.wide_space(d, n_tasks=2, n=n, d=d, ks=ks, n_iter=5, card_wide=(64, 2048))
    corners = rng.choice([0, 2047], size=(12, d))
    for t in range(2):
        rows = wl.task_rows(t)
        rows[:] = corners[rng.integers(0, 12, size=n)]
        noise = rng.integers(0, 200, size=rows.shape)
        rows[:] = np.where(rows > 1000, rows - noise, rows + noise)
        if t == 1:
            rows[0] = 1000                           # a first row (the first start) away from all others
    wl.cards[:] = 2048
    _sweep(wl, flags=binding.F_VALUES_BELOW_2048, sfx="_u16", want_trace=True)


@pytest.mark.parametrize("d", [40, 47])
def test_most_rows_on_the_far_side_of_the_first_ones(d):
    # every centroid moves to one side of the offset (the mean of the starts), a few rows stay on the other
    rng = np.random.default_rng(d + 1)
    wl = workloads.wide_space(d, n_tasks=1, n=1500, d=d, ks=(1, 2, 4), n_iter=5, card_wide=(64, 2048))
    rows = wl.rows
    rows[:] = 1900 + rng.integers(0, 100, size=rows.shape)
    rows[:8] = 1000 + rng.integers(0, 60, size=(8, d))
    rows[50:60] = rng.integers(0, 40, size=(10, d))
    wl.cards[:] = 2048
    _sweep(wl, flags=binding.F_VALUES_BELOW_2048, sfx="_u16")


def _all_far(wl, far, same_norm):
    # nothing near the rows; with equal norms the order of two starts hangs on x . mu alone
    rng = np.random.default_rng(wl.n_total)
    shape = (wl.T, sum(wl.ks), wl.d)
    size = far if same_norm else far * (1.0 + rng.random(shape[:2]))[:, :, None]
    return 128.0 + size * rng.choice([-1.0, 1.0], size=shape)


@pytest.mark.parametrize("same_norm", [True, False])
@pytest.mark.parametrize("far", [1e8, 3e15, 1e16, 1e18, 1e25, 1e200])
@pytest.mark.parametrize("d,n,ks", [(9, 700, (3, 31, 63)), (16, 641, (40, 70)), (24, 900, (5, 33))])
def test_streaming_starts_beyond_the_padding_scores(d, n, ks, far, same_norm):
    # an unclamped |mu'|^2 exceeds the score of padding rows, and its rounding the bound under which every centroid is a candidate
    wl = workloads.random_task(n, n, d, card_lo=100, card_hi=256, n_blobs=9, sigma=30.0, ks=ks, n_iter=3, n_tasks=2)
    _sweep(wl, init=_all_far(wl, far, same_norm), flags=binding.F_STREAMING, path=1)


@pytest.mark.parametrize("same_norm", [True, False])
@pytest.mark.parametrize("far", [1e8, 3e15, 1e16, 1e18, 1e25, 1e200])
@pytest.mark.parametrize("d,n,ks", [(7, 700, (3, 31, 63)), (32, 1100, (8, 64)), (45, 600, (5, 30))])
def test_two_part_starts_beyond_the_padding_scores(d, n, ks, far, same_norm):
    import torch
    wl = workloads.wide_space(n + d, n_tasks=2, n=n, d=d, ks=ks, n_iter=3, card_wide=(64, 9000))
    init = _all_far(wl, far, same_norm)
    dw = binding.DeviceWorkload(wl)
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off, wl.ks, wl.n_iter, init_centroids=torch.from_numpy(init).to(dw.X.device), want_labels=True,
                                    _sfx="_u16")
    check_sweep(wl, out, oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, init=init, want_labels=True), dw.ld)
