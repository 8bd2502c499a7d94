"""The order in which a loss is summed belongs to the task, its k and the largest task of the batch: it is the same in a whole
sweep, in any chunking of it, with or without a trace, and (streaming path) whatever else is in the batch.  The knee rule compares
these sums, so they are compared bit for bit here."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads

pytestmark = pytest.mark.gpu


def _wave_sum(v):
    """64 lanes, partner lane ^ 32, 16, ..., 1."""
    lanes = np.arange(64)
    for off in (32, 16, 8, 4, 2, 1):
        v = v + v[lanes ^ off]
    return v[0]


def _streaming_loss(rows, labels, mu, k):
    """Blocks of 4096 rows; in a block four waves take runs of 128 rows in turn (256 with at most 16 knobs and k <= 64), 64 rows
    at a time; waves, then blocks, in order."""
    d = rows.shape[1]
    term = np.zeros(len(rows))
    for j in range(d):
        t = rows[:, j].astype(np.float64) - mu[labels, j]
        term = term + t * t
    run = 256 if d <= 16 and k <= 64 else 128
    total = 0.0
    for b in range(0, len(rows), 4096):
        block = np.zeros(4096)
        n = min(4096, len(rows) - b)
        block[:n] = term[b:b + n]
        steps = block.reshape(4096 // (4 * run), 4, run // 64, 64)
        s = 0.0
        for w in range(4):
            part = np.zeros(64)
            for i in range(steps.shape[0]):
                for q in range(run // 64):
                    part = part + steps[i, w, q]
            s = s + _wave_sum(part)
        total = total + s
    return total


def _streaming(dw, off, wl, **kw):
    return binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, off, wl.ks, wl.n_iter, flags=binding.F_STREAMING, **kw)


@pytest.mark.parametrize("n,d,ks", [(1, 5, (1,)), (513, 16, (3, 64, 65)), (4095, 17, (2, 40)), (4096, 9, (7, 100)), (4097, 24, (5, 33, 256)),
                                    (12289, 16, (16, 80)), (30001, 31, (2, 64))])
def test_streaming_loss_is_the_documented_sum(n, d, ks):
    wl = workloads.random_task(n + d, n, d, card_hi=30, n_blobs=7, sigma=1.1, ks=ks, n_iter=4, n_tasks=2, ragged=n > 1)
    dw = binding.DeviceWorkload(wl)
    out = _streaming(dw, wl.task_off, wl, want_labels=True)
    traced = _streaming(dw, wl.task_off, wl, want_trace=True)
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, want_labels=True)
    got = out["inertia"].cpu().numpy()
    np.testing.assert_array_equal(traced["inertia"].cpu().numpy(), got)
    np.testing.assert_array_equal(traced["trace"].cpu().numpy()[:, :, -1], got)
    for t in range(2):
        rows = slice(wl.task_off[t], wl.task_off[t + 1])
        for i, k in enumerate(ks):
            if ref["status"][t, i] == 0:
                mu = ref["centroids"][t, ref["koff"][i]:ref["koff"][i + 1]]
                assert got[t, i] == _streaming_loss(wl.rows[rows], ref["labels"][i, rows], mu, k), (t, k)
            else:
                assert got[t, i] == 0.0


@pytest.mark.parametrize("n,d", [(700, 9), (5000, 14), (9000, 24)])
def test_streaming_loss_does_not_depend_on_the_batch(n, d):
    # alone a task's rows are split over the chip, among 60 others a workgroup takes them all
    wl = workloads.random_task(n, n, d, card_hi=20, n_blobs=6, sigma=0.9, ks=(2, 9, 40, 70), n_iter=5, n_tasks=60, ragged=True)
    dw = binding.DeviceWorkload(wl)
    whole = _streaming(dw, wl.task_off, wl)["inertia"].cpu().numpy()
    for t in (0, 17, 59):
        alone = _streaming(dw, wl.task_off[t:t + 2], wl)["inertia"].cpu().numpy()
        np.testing.assert_array_equal(alone[0], whole[t])


def _chunked_equals_whole(wl, chunk, flags, sfx="", path=None):
    dw = binding.DeviceWorkload(wl)
    assert binding.cham_sweep_path(dw.ld, dw.d, wl.task_off, wl.ks, flags=flags, _sfx=sfx) == path
    whole = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, flags=flags, _sfx=sfx)
    part = binding.cham_kmeans_sweep_knee(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, threshold=0.0, chunk=chunk, flags=flags, _sfx=sfx)
    for key in ("status", "counts", "centroids", "inertia"):
        np.testing.assert_array_equal(part[key].cpu().numpy(), whole[key].cpu().numpy(), err_msg=key)


@pytest.mark.parametrize("n,d,tasks", [(5000, 14, 40), (6000, 24, 60), (9000, 9, 30), (120000, 12, 3)])
@pytest.mark.parametrize("chunk", [1, 3])
def test_chunked_streaming_sweep(n, d, tasks, chunk):
    wl = workloads.random_task(n + d, n, d, card_hi=18, n_blobs=6, sigma=0.9, ks=(2, 4, 8, 16, 32, 64, 128), n_iter=4, n_tasks=tasks, ragged=True)
    _chunked_equals_whole(wl, chunk, binding.F_STREAMING, path=1)


@pytest.mark.parametrize("n_iter", [3, 40])
@pytest.mark.parametrize("n,d,tasks,ks,chunk", [(500, 12, 40, range(2, 12), 3), (1800, 24, 20, range(8, 41), 5)])
def test_chunked_resident_sweep(n, d, tasks, ks, chunk, n_iter):
    # the whole list has units for more than every place of the chip, a chunk of it has not: the rows of a task are split over the
    # waves in another way.  n_iter = 3: units that have not reached their fixed point.
    wl = workloads.random_task(n, n, d, card_hi=24, n_blobs=9, sigma=1.2, ks=tuple(ks), n_iter=n_iter, n_tasks=tasks, ragged=True)
    _chunked_equals_whole(wl, chunk, 0, path=0)
    wl = workloads.wide_space(n, n_tasks=tasks, n=n, d=d, ks=tuple(ks), n_iter=n_iter, ragged=True)
    _chunked_equals_whole(wl, chunk, binding.F_VALUES_BELOW_2048, sfx="_u16", path=0)


@pytest.mark.parametrize("n,d,flags,path", [(1000, 32, 0, 0), (2000, 32, 0, 0), (2000, 32, binding.F_NO_MFMA, 2)])
def test_chunked_sweep_of_all_byte_knobs(n, d, flags, path):
    wl = workloads.random_task(n, n, d, card_hi=24, n_blobs=9, sigma=1.2, ks=tuple(range(2, 34, 3)), n_iter=3, n_tasks=30, ragged=True)
    _chunked_equals_whole(wl, 2, flags, path=path)


@pytest.mark.parametrize("n,d", [(900, 40), (2048, 47), (1500, 60)])
def test_chunked_sweep_of_two_byte_knobs(n, d):
    # rows of 48 and of 64 slots
    wl = workloads.wide_space(n, n_tasks=20, n=n, d=d, ks=tuple(range(2, 32)), n_iter=3, ragged=True)
    _chunked_equals_whole(wl, 4, binding.F_VALUES_BELOW_2048, sfx="_u16", path=0)


@pytest.mark.parametrize("n,d,ks", [(500, 12, (2, 9, 33)), (2000, 24, tuple(range(2, 42)))])
def test_resident_loss_does_not_depend_on_the_batch(n, d, ks):
    # (the largest task of a batch sets the number of waves: tasks of one size)
    wl = workloads.random_task(n, n, d, card_hi=24, n_blobs=9, sigma=1.2, ks=ks, n_iter=4, n_tasks=100)
    dw = binding.DeviceWorkload(wl)
    whole = binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off, ks, wl.n_iter, want_trace=True)
    for t in (0, 99):
        alone = binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off[t:t + 2], ks, wl.n_iter, want_trace=True)
        for key in ("inertia", "trace"):
            np.testing.assert_array_equal(alone[key][0].cpu().numpy(), whole[key][t].cpu().numpy())


def _subset_has_the_whole_batchs_losses(wl, ks, n_iter, flags, sfx):
    """Two tasks next to each other, the largest of the batch among them: few units, another form of the kernel."""
    dw = binding.DeviceWorkload(wl)
    off = np.asarray(wl.task_off)
    whole = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, off, ks, n_iter, want_trace=True, flags=flags, _sfx=sfx)
    plain = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, off, ks, n_iter, flags=flags, _sfx=sfx)
    big = int(np.argmax(np.diff(off)))
    for t in {max(0, big - 1), min(big, wl.T - 2)}:
        two = off[t:t + 3]
        alone = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, two, ks, n_iter, want_trace=True, flags=flags, _sfx=sfx)
        quiet = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, two, ks, n_iter, flags=flags, _sfx=sfx)
        for key in ("status", "counts", "centroids", "inertia", "trace"):
            np.testing.assert_array_equal(alone[key].cpu().numpy(), whole[key][t:t + 2].cpu().numpy(), err_msg=key)
        np.testing.assert_array_equal(quiet["inertia"].cpu().numpy(), plain["inertia"][t:t + 2].cpu().numpy())


@pytest.mark.parametrize("n_iter", [3, 30])
@pytest.mark.parametrize("n", [1025, 1300, 1537, 2048])
def test_loss_of_all_byte_knobs_does_not_depend_on_the_batch(n, n_iter):
    wl = workloads.random_task(n, n, 32, card_hi=24, n_blobs=9, sigma=1.2, ks=(2, 9, 33, 50), n_iter=n_iter, n_tasks=80, ragged=True)
    _subset_has_the_whole_batchs_losses(wl, wl.ks, n_iter, 0, "")


@pytest.mark.parametrize("n_iter", [3, 30])
@pytest.mark.parametrize("n,d", [(513, 40), (700, 33), (900, 47), (1024, 48), (1000, 63)])
def test_loss_of_many_two_byte_knobs_does_not_depend_on_the_batch(n, d, n_iter):
    wl = workloads.wide_space(n, n_tasks=80, n=n, d=d, ks=(2, 9, 32), n_iter=n_iter, ragged=True)
    # (ragged sizes: the largest task stays above 512 rows)
    off = np.asarray(wl.task_off)
    if np.diff(off).max() <= 512:
        wl = workloads.wide_space(n, n_tasks=80, n=n, d=d, ks=(2, 9, 32), n_iter=n_iter)
    _subset_has_the_whole_batchs_losses(wl, wl.ks, n_iter, binding.F_VALUES_BELOW_2048, "_u16")


def _loss_errors(wl, out):
    """|loss - exact| / exact, the exact one in 80-bit arithmetic from the sweep's own labels and centroids."""
    lab, cen, got = (out[key].cpu().numpy() for key in ("labels", "centroids", "inertia"))
    koff = np.concatenate([[0], np.cumsum(wl.ks)])
    err = []
    for t in range(wl.T):
        r = slice(wl.task_off[t], wl.task_off[t + 1])
        x = wl.rows[r].astype(np.longdouble)
        for i in range(len(wl.ks)):
            exact = ((x - cen[t, koff[i]:koff[i + 1]].astype(np.longdouble)[lab[i, r]]) ** 2).sum()
            err.append(float(abs(got[t, i] - exact) / exact))
    return np.array(err)


def test_losses_of_values_in_two_parts_are_as_exact_as_the_vector_kernels():
    # Both sum doubles; what differs is the depth of the sums.  Means over 576 losses: 6.4e-17 against the vector kernel's 7.3e-17 with the
    # sixteen parts of a task added pairwise, 8.5e-17 with one after the other.  (The standard error of such a mean is 3 %.)
    here, vector = [], []
    for d, n, n_iter, top in ((17, 700, 20, 8000), (27, 1900, 20, 60000), (40, 1900, 4, 9000)):
        wl = workloads.wide_space(d + n, n_tasks=48, n=n, d=d, ks=(4, 12, 20, 32), n_iter=n_iter, card_wide=(64, top), ragged=True)
        dw = binding.DeviceWorkload(wl)
        assert binding.cham_sweep_kernel_u16(dw.ld, d, wl.task_off, wl.ks) == "resident_mfma_kernel"
        for flags, errors in ((0, here), (binding.F_NO_MFMA, vector)):
            out = binding.cham_kmeans_sweep(dw.X, dw.ld, d, wl.task_off, wl.ks, n_iter, want_labels=True, flags=flags, _sfx="_u16")
            errors.append(_loss_errors(wl, out))
    assert np.concatenate(here).mean() <= 1.03 * np.concatenate(vector).mean()
