"""Lookups by groups of eight lanes and wave-wide modes of the synthesis kernels: sizes of the visited set around
the nine-way split, histograms of one word and of several windows, more flagged clusters than fit a round."""
import numpy as np
import pytest

from paper_2001_08743_amd import workloads
from parity_util import check_pipeline, check_sweep, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_visited", [1, 2, 8, 9, 10, 80, 81, 82, 731])
@pytest.mark.parametrize("n,k", [(300, 7), (2300, 200), (17000, 65)])
def test_lookup_in_small_visited_sets(n, k, n_visited):
    # n = 17000: the variant that splits a task over several workgroups; k = 200: more than 128 lookups at once
    wl = workloads.random_task(100 * n_visited + k, n, 9, card_lo=1, card_hi=12, n_blobs=5, invalid_frac=0.2, ks=(2, k), n_iter=3,
                               n_visited=n_visited)
    _, g, c = run_both(wl, threshold=0.0)           # never at the knee: the largest k is chosen
    check_sweep(wl, g["sweep"], c, (wl.n_total + 63) // 64 * 64)
    assert int(g["chosen"].cpu().numpy()[0]) == 1
    check_pipeline(wl, g, c)


@pytest.mark.parametrize("card_wide", [(2, 3), (63, 65), (9000, 16384)])
def test_modes_of_two_byte_knobs_by_waves(card_wide):
    wl = workloads.wide_space(card_wide[1], n_tasks=3, n=700, d=11, ks=(3, 17), n_iter=3, n_visited=64, wide_frac=0.5, card_wide=card_wide,
                              card_small=(1, 4), ragged=True)
    wl.valid[: wl.n_total // 2] = 0                  # clusters without a valid member among them
    _, g, c = run_both(wl, threshold=0.0)
    check_pipeline(wl, g, c)
    flags = g["synth"]["out_flag"].cpu().numpy()
    assert np.isin(flags, (2, 3)).any()
