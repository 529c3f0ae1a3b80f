"""Every width of the sorted merge (a level needs D-s+1 entries, rounded up to a multiple of eight),
every level of a search as deep as its device count, on both forms of the level kernel and both value
widths, and the recomputed stage times of 64-bit values at the bound of their exact range."""
import numpy as np
import pytest

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match, assert_tables_match, gpu_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo", [B.ALGO_MERGE, B.ALGO_RECOMPUTE])
@pytest.mark.parametrize("width", [B.NARROW_MAX_TOTAL_TIME, B.WIDE_RECOMPUTE_MAX_TOTAL_TIME])
@pytest.mark.parametrize("D", [2, 8, 9, 16, 17, 24, 25, 33, 40, 41, 49, 57, 64])
def test_every_level_of_a_deep_search(D, width, algo):
    probs = [synth.random_small(40 + D, 66, D, D, tight=1.5, tmax=10**6),
             synth.random_small(41 + D, 65, max(2, D - 3), D, tight=40.0, tmax=3)]
    for group in (probs[:1], probs):   # descriptor as a kernel argument, and an array of them
        res, sess = gpu_run(group, max_total_time_ns=width, algo=algo, one_launch_small=1)
        with sess:
            rc, info = B.rannc_dp_solve_info(sess.h)
            want = B.KERNEL_MERGE_RECOMPUTE if algo == B.ALGO_RECOMPUTE else B.KERNEL_MERGE_TABLE
            assert all(info.level_kernel[k] == want for k in range(4) if info.n_problems[k])
            assert_results_match(group, res)
            for q in range(len(group)):
                assert_tables_match(group[q], sess, q, args=False)


@pytest.mark.parametrize("N", [64, 65, 97, 129, 200])
def test_recomputed_64_bit_stage_times_up_to_their_bound(N):
    top = B.WIDE_RECOMPUTE_MAX_TOTAL_TIME
    g = np.random.default_rng(N)
    probs = []
    for case, D in enumerate((7, 31, 48, 64)):
        pr = synth.random_small(60 + case, N, D, min(D, 9), tight=(1.4, 60.0)[case % 2], tmax=9)
        t = g.integers(0, 1 << 31, N).astype(np.int64)
        t[int(g.integers(0, N))] += top - int(t.sum())     # the whole chain is exactly the bound
        pr["time_ns"] = t
        probs.append(pr)
    for rows in (0, 1, 16):
        res, sess = gpu_run(probs, max_total_time_ns=top, algo=B.ALGO_RECOMPUTE, one_launch_small=1, rows_per_wave=rows)
        with sess:
            assert_results_match(probs, res)
            for q in range(len(probs)):
                assert_tables_match(probs[q], sess, q, args=False)
