"""Two-byte knobs without the promise on the matrix cores (values in two f16 parts): sizes around its limits, values up to 65535, starts
far outside the range, ties, against the oracle and bit for bit against the vector kernel."""
import numpy as np
import pytest

import oracle
from paper_2001_08743_amd import binding, workloads
from parity_util import check_sweep

pytestmark = pytest.mark.gpu


def _sweep(wl, init=None, want_trace=False):
    import torch
    dw = binding.DeviceWorkload(wl)
    in_two_parts = int(np.diff(wl.task_off).max()) > 256       # (a ragged batch of nominally 257 rows stays on the vector kernel)
    assert binding.cham_sweep_kernel_u16(dw.ld, dw.d, wl.task_off, wl.ks) == ("resident_mfma_kernel" if in_two_parts else "resident_sweep_kernel")
    kw = {} if init is None else dict(init_centroids=torch.from_numpy(init).to(dw.X.device))
    out = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, want_trace=want_trace, _sfx="_u16", **kw)
    vec = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, flags=binding.F_NO_MFMA, _sfx="_u16", **kw)
    torch.cuda.synchronize()
    for key in ("status", "counts", "centroids", "labels"):
        n = wl.n_total if key == "labels" else None
        a, b = out[key].cpu().numpy(), vec[key].cpu().numpy()
        np.testing.assert_array_equal(a[:, :n] if n else a, b[:, :n] if n else b, err_msg=key)
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, init=init, want_labels=True, want_trace=want_trace)
    check_sweep(wl, out, ref, dw.ld)


@pytest.mark.parametrize("n", [257, 1023, 1900, 2048])
@pytest.mark.parametrize("d,ks", [(5, (2, 8, 64)), (16, (9, 33)), (27, (3, 32)), (32, (17, 40)), (33, (8, 32)), (48, (5, 31))])
def test_sizes(n, d, ks):
    wl = workloads.wide_space(n + d, n_tasks=3, n=n, d=d, ks=ks, n_iter=9, card_wide=(64, 8000), ragged=n % 2 == 1)
    _sweep(wl, want_trace=n == 257)


@pytest.mark.parametrize("n,d,ks", [(4096, 20, (8, 50)), (3001, 32, (64,)), (2049, 32, (12,))])
def test_tasks_beyond_2048_rows(n, d, ks):
    wl = workloads.wide_space(n + d, n_tasks=2, n=n, d=d, ks=ks, n_iter=6, card_wide=(64, 20000), ragged=False)
    _sweep(wl)


@pytest.mark.parametrize("d", [11, 32, 47])
@pytest.mark.parametrize("values", [(0, 65535), (65279, 65280, 65535), (0, 255, 256, 257, 32767, 32768), (7, 8, 9)])
def test_extreme_values(d, values):
    # few values: rows at equal distances from several centroids, both ends of the range, the steps of the parts
    rng = np.random.default_rng(d + len(values))
    wl = workloads.wide_space(d, n_tasks=2, n=700, d=d, ks=(8, 20), n_iter=5, card_wide=(64, 600))
    wl.rows[:] = rng.choice(np.array(values, dtype=np.int64), size=wl.rows.shape).astype(wl.rows.dtype)
    _sweep(wl)


@pytest.mark.parametrize("far", [1.0e5, 3.0e5, 1.0e9])
def test_far_starts(far):
    wl = workloads.wide_space(3, n_tasks=2, n=600, d=21, ks=(10,), n_iter=4, card_wide=(64, 60000))
    init = np.tile(wl.rows[:10].astype(np.float64), (2, 1, 1)).reshape(2, 10, 21)
    init[:, 4:] += far * np.arange(1, 7)[None, :, None]
    init[:, 5, 3] = -far
    _sweep(wl, init=init)


@pytest.mark.parametrize("chunk", [1, 3])
def test_chunked_sweep_equals_the_whole(chunk):
    wl = workloads.wide_space(9, n_tasks=20, n=1500, d=24, ks=tuple(range(2, 30, 2)), n_iter=3, card_wide=(64, 5000), ragged=True)
    dw = binding.DeviceWorkload(wl)
    whole = binding.cham_kmeans_sweep(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, _sfx="_u16")
    part = binding.cham_kmeans_sweep_knee(dw.X, dw.ld, dw.d, wl.task_off, wl.ks, wl.n_iter, threshold=0.0, chunk=chunk, _sfx="_u16")
    for key in ("status", "counts", "centroids", "inertia"):
        np.testing.assert_array_equal(part[key].cpu().numpy(), whole[key].cpu().numpy(), err_msg=key)


@pytest.mark.parametrize("d", [31, 32, 33])
@pytest.mark.parametrize("flags", [0, binding.F_VALUES_BELOW_2048])
def test_many_tiny_tasks_beside_a_large_one(d, flags):
    # every task takes a tile of its own in the packed copies, whatever its rows
    wl = workloads.wide_space(d, n_tasks=1, n=300 * 3 + 1100, d=d, ks=(2, 8), n_iter=6, card_wide=(64, 2000))
    wl.task_off = np.concatenate([np.arange(0, 901, 3), [2000]]).astype(np.int64)
    import torch
    X = torch.zeros((d, 2048), dtype=torch.int16, device="cuda")
    X[:, :2000] = torch.from_numpy(np.ascontiguousarray(wl.rows.T).view(np.int16)).cuda()
    out = binding.cham_kmeans_sweep(X, 2048, d, wl.task_off, wl.ks, wl.n_iter, want_labels=True, flags=flags, _sfx="_u16")
    torch.cuda.synchronize()
    ref = oracle.sweep(wl.rows, wl.task_off, wl.ks, wl.n_iter, want_labels=True)
    np.testing.assert_array_equal(out["status"].cpu().numpy(), ref["status"])
    np.testing.assert_array_equal(out["counts"].cpu().numpy(), ref["counts"])
    np.testing.assert_array_equal(out["centroids"].cpu().numpy(), ref["centroids"])


@pytest.mark.parametrize("n,d,ks", [(257, 5, (2, 24)), (257, 16, (8,)), (257, 32, (3, 64)), (257, 48, (5, 32)), (1025, 8, (33,)), (1025, 16, (16,)), (4096, 17, (8, 64)),
                                    (2048, 33, (8,))])
def test_edges_of_the_rule(n, d, ks):
    wl = workloads.wide_space(n + d, n_tasks=2, n=n, d=d, ks=ks, n_iter=7, card_wide=(64, 8000), ragged=False)
    assert int(np.diff(wl.task_off).max()) == n
    _sweep(wl, want_trace=True)
