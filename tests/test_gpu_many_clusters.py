"""Lists of k beyond 64 without a flag: the resident matrix-core kernel's form for many centroids, up to k = 224 and 7000 rows x chunks of 64
centroids, and the streaming kernels behind that.  Sizes around the chunks, the waves' rows, the LDS limits and the limit
between the two, against the oracle; losses of chunks of the list against the whole list's."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import check_sweep

pytestmark = pytest.mark.gpu


def _sweep(wl, want_trace=False, init=None):
    import torch
    dw = binding.DeviceWorkload(wl)
    resident = max(wl.ks) <= 224 and int(np.diff(wl.task_off).max()) * -(-max(wl.ks) // 64) <= 7000
    assert binding.cham_sweep_kernel(dw.ld, dw.d, wl.task_off, wl.ks) == ("resident_mfma_kernel" if resident else "stream_assign_kernel")
    kw = {} if init is None else dict(init_centroids=torch.from_numpy(init).to(dw.X.device))
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=want_trace, **kw)
    torch.cuda.synchronize()
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, init=init, want_labels=True, want_trace=want_trace)
    check_sweep(wl, out, ref, dw.ld)
    return dw, out


@pytest.mark.parametrize("n", [66, 300, 1023, 1025, 1749, 1751, 2333, 2334, 3499, 3501, 4096])
@pytest.mark.parametrize("d,ks", [(9, (5, 64, 65)), (15, (96, 97, 128)), (16, (33, 129, 160)), (24, (2, 191, 192)), (31, (193, 224))])
def test_sizes(n, d, ks):
    wl = workloads.random_task(3 * n + d, n, d, card_hi=20, n_blobs=9, sigma=0.8, ks=ks, n_iter=12, n_tasks=3, ragged=n % 2 == 1)
    _sweep(wl, want_trace=n == 300)


@pytest.mark.parametrize("k", [100, 200])
def test_ties_on_every_row(k):
    # few values per knob: many rows at the same distance from several centroids, more (row, candidate) pairs than a queue holds
    wl = workloads.random_task(k, 1500, 8, card_hi=3, n_blobs=3, sigma=2.0, ks=(k,), n_iter=6, n_tasks=2)
    _sweep(wl)


def test_candidates_without_number():
    # starts far outside the knobs' range: every centroid is a candidate of every row
    wl = workloads.random_task(5, 700, 12, card_hi=12, n_blobs=5, sigma=1.0, ks=(70,), n_iter=3, n_tasks=2)
    init = np.full((2, 70, 12), 1.0e9) + np.arange(70)[None, :, None]
    init[:, :3] = wl.rows[:3].astype(np.float64)
    _sweep(wl, init=init)


def test_unaligned_tasks_and_more_units_than_places():
    wl = workloads.random_task(6, 333, 10, card_hi=16, n_blobs=6, sigma=0.8, ks=tuple(range(60, 74)), n_iter=8, n_tasks=30, ragged=True)
    _sweep(wl)


@pytest.mark.parametrize("chunk", [1, 2])
def test_chunked_sweep_equals_the_whole(chunk):
    wl = workloads.random_task(7, 2000, 14, card_hi=18, n_blobs=6, sigma=0.9, ks=(8, 64, 65, 128, 130), n_iter=3, n_tasks=9, ragged=True)
    dw, whole = _sweep(wl)
    part = binding.cham_kmeans_sweep_knee(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, threshold=0.0, chunk=chunk, want_labels=True)
    for key in ("status", "counts", "centroids", "labels", "inertia"):
        np.testing.assert_array_equal(part[key].cpu().numpy(), whole[key].cpu().numpy(), err_msg=key)


def _far_starts(wl, ks, far):
    # every start outside the range of the screen's operands (some 2300 from the rows), so that every score is within the bound
    rng = np.random.default_rng(wl.n_total)
    return 128.0 + far * (1.0 + 0.1 * rng.random((wl.T, sum(ks), 1))) * rng.choice([-1.0, 1.0], size=(wl.T, sum(ks), wl.d))


@pytest.mark.parametrize("far", [5.0e3, 1.0e6])
@pytest.mark.parametrize("d", [9, 24])
@pytest.mark.parametrize("n,k", [(65, 70), (130, 70), (641, 70), (642, 70), (641, 100), (642, 100), (641, 129), (1281, 193)])
def test_candidates_without_number_listed_pair_by_pair(n, k, d, far):
    # the last wave owns one or two rows: their candidates fit the list of pairs, which holds no centroid beyond k
    wl = workloads.random_task(n + d, n, d, card_lo=100, card_hi=256, n_blobs=9, sigma=20.0, ks=(k,), n_iter=2, n_tasks=2)
    _sweep(wl, init=_far_starts(wl, (k,), far))


@pytest.mark.parametrize("byte", [0x00, 0xFF, 0x40])
@pytest.mark.parametrize("d", [9, 24])
@pytest.mark.parametrize("n,k", [(65, 70), (641, 70), (642, 100), (641, 129), (641, 250)])
def test_streaming_candidates_without_number_listed_pair_by_pair(n, k, d, byte):
    # ... whatever the workspace held before
    import torch
    wl = workloads.random_task(n + d, n, d, card_lo=100, card_hi=256, n_blobs=9, sigma=20.0, ks=(k,), n_iter=2, n_tasks=2)
    init = _far_starts(wl, (k,), 1.0e5)
    dw = binding.DeviceWorkload(wl)
    size = binding.cham_sweep_workspace_bytes(dw.ld, d, wl.task_off, wl.ks, wl.n_iter, binding.F_STREAMING)
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off, wl.ks, wl.n_iter, init_centroids=torch.from_numpy(init).to(dw.X.device), want_labels=True,
                                    flags=binding.F_STREAMING, workspace=torch.full((size,), byte, dtype=torch.uint8, device=dw.X.device))
    torch.cuda.synchronize()
    check_sweep(wl, out, oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, init=init, want_labels=True), dw.ld)


@pytest.mark.parametrize("n,d,k", [(641, 9, 70), (1500, 24, 100), (2333, 15, 129), (1281, 31, 193)])
@pytest.mark.parametrize("near", [0, 1, 40])
def test_starts_no_row_can_be_nearest_to(n, d, k, near):
    # from three times the farthest row's (or the nearest start's) distance on a start takes no part in the screen: starts on both sides of that, from
    # just outside the rows to 1e200, centroid 0 among them, with none, one and many starts among the rows
    wl = workloads.random_task(n + d + near, n, d, card_lo=100, card_hi=256, n_blobs=9, sigma=20.0, ks=(64, k), n_iter=6, n_tasks=2)
    rng = np.random.default_rng(n)
    away = np.concatenate([np.geomspace(0.8, 4.0, 24), np.geomspace(10.0, 1.0e4, 12), [1.0e9, 1.0e17, 1.0e200]])
    init = np.empty((2, 64 + k, d))
    for t in range(2):
        rows = wl.rows[wl.task_off[t]:wl.task_off[t + 1]].astype(np.float64)
        centre = rows.mean(axis=0)
        reach = np.sqrt(((rows - centre) ** 2).sum(axis=1).max())
        way = rng.normal(size=(64 + k, d))
        init[t] = centre + way / np.linalg.norm(way, axis=1, keepdims=True) * reach * rng.choice(away, size=(64 + k, 1))
        for first, kk in ((0, 64), (64, k)):
            init[t, first + kk - near:first + kk] = rows[:near]
    _sweep(wl, want_trace=True, init=init)
    import torch
    dw = binding.DeviceWorkload(wl)
    both = [binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off, wl.ks, wl.n_iter, init_centroids=torch.from_numpy(init).to(dw.X.device), want_labels=True, flags=f)
            for f in (0, binding.F_STREAMING)]
    _same_bits(*both, ("status", "centroids", "counts", "inertia"))


def _same_bits(a, b, keys):
    for key in keys:
        np.testing.assert_array_equal(a[key].cpu().numpy(), b[key].cpu().numpy(), err_msg=key)


@pytest.mark.parametrize("n_iter", [2, 25])
@pytest.mark.parametrize("n,d,ks", [(65, 5, (65,)), (300, 15, (3, 64, 65)), (1025, 16, (40, 100)), (2333, 17, (64, 150)), (3499, 16, (30, 128)), (1750, 31, (9, 224)),
                                    (3500, 24, (63, 65))])
def test_loss_is_that_of_the_streaming_kernels(n, d, ks, n_iter):
    # the knee rule compares losses: they belong to a task and its k, whichever of the two forms the batch runs on, with and without a trace,
    # at the fixed point or not
    wl = workloads.random_task(n + d, n, d, card_hi=30, n_blobs=7, sigma=1.1, ks=ks, n_iter=n_iter, n_tasks=2, ragged=True)
    dw = binding.DeviceWorkload(wl)
    sweep = lambda **kw: binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off, ks, n_iter, **kw)
    plain, traced, streamed = sweep(), sweep(want_trace=True), sweep(want_trace=True, flags=binding.F_STREAMING)
    _same_bits(plain, streamed, ("status", "centroids", "counts", "inertia"))
    _same_bits(traced, streamed, ("inertia", "trace"))


def test_loss_does_not_depend_on_the_batch():
    wl = workloads.random_task(11, 4096, 14, card_hi=18, n_blobs=6, sigma=0.9, ks=(8, 65, 130), n_iter=3, n_tasks=6, ragged=True)
    off = wl.task_off
    dw = binding.DeviceWorkload(wl)
    whole = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, off, wl.ks, wl.n_iter)["inertia"].cpu().numpy()
    sizes = np.diff(off)
    assert sizes.max() * 3 > 7000 > sizes.min() * 3         # together they stream, the smaller ones alone do not
    for t in range(wl.T):
        alone = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, off[t:t + 2], wl.ks, wl.n_iter)["inertia"].cpu().numpy()
        np.testing.assert_array_equal(alone[0], whole[t])


def test_loss_of_tasks_without_rows():
    import torch
    wl = workloads.random_task(12, 200, 6, card_hi=9, n_blobs=3, sigma=1.0, ks=(66,), n_iter=2, n_tasks=2)
    off = np.array([0, 0, 3, 3, 200], dtype=np.int64)
    dw = binding.DeviceWorkload(wl)
    init = np.random.default_rng(1).uniform(0, 9, size=(4, 66, 6))
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, 6, off, wl.ks, 2, init_centroids=torch.from_numpy(init).to(dw.X.device))
    ref = oracle.sweep(wl.rows[:200], off, wl.ks, 2, init=init)
    np.testing.assert_allclose(out["inertia"].cpu().numpy(), ref["inertia"], rtol=1e-12, atol=0)
    np.testing.assert_array_equal(out["counts"].cpu().numpy(), ref["counts"])
