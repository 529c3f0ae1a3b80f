"""Work items of the recomputing level kernel inside the diagonal block of a chunk, on 64-bit values: short
segments (a last chunk of 18 to 32 rows, or a window that starts inside the block because the chunk's first
block fits no device) in items as large as the list allows."""
import numpy as np
import pytest
import torch

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match, assert_tables_match, gpu_run, oracle_solve_many

pytestmark = pytest.mark.gpu
TOP = B.WIDE_RECOMPUTE_MAX_TOTAL_TIME


def _chain(seed, N, D, S, oversized=None):
    pr = synth.random_small(seed, N, D, S, tight=2.5, tmax=10**6)
    pr["time_ns"] = pr["time_ns"] * 1000
    if oversized is not None:
        pr["param_bytes"] = pr["param_bytes"].copy()
        pr["param_bytes"][oversized] = pr["mem_capacity"] + 1
    return pr


@pytest.mark.parametrize("rows", [0, 8, 16])
@pytest.mark.parametrize("N,oversized", [(82, None), (95, None), (96, 64), (150, None), (160, 128), (190, 64), (222, None)])
def test_short_diagonal_segments(N, oversized, rows):
    probs = [_chain(N + D, N, D, 4, oversized) for D in (64, 31)]
    for group in (probs[:1], probs):
        res, sess = gpu_run(group, max_total_time_ns=TOP, algo=B.ALGO_RECOMPUTE, one_launch_small=1, rows_per_wave=rows)
        with sess:
            rc, info = B.rannc_dp_solve_info(sess.h)
            assert {info.level_kernel[k] for k in range(4) if info.n_problems[k]} == {B.KERNEL_MERGE_RECOMPUTE}
            assert_results_match(group, res)
            for q in range(len(group)):
                assert_tables_match(group[q], sess, q, args=False)


def test_batch_that_takes_the_largest_items():
    probs = [_chain(3000 + q, 160, 64, 3, 128 if q % 16 == 7 else None) for q in range(128)]
    res, sess = gpu_run(probs, max_total_time_ns=TOP)
    with sess:
        rc, info = B.rannc_dp_solve_info(sess.h)
        assert info.level_kernel[3] == B.KERNEL_MERGE_RECOMPUTE
        assert_results_match(probs, res, oracle_results=oracle_solve_many(probs))
        for q in (0, 7, 127):
            assert_tables_match(probs[q], sess, q, args=False)


@pytest.mark.parametrize("N", [1234, 1300])
def test_large_search_equals_the_table_form(N):
    pr = synth.enlarged_transformer_chain(seed=5, N=N, D=64, S=4, MB=64, M=1 << 40)
    rr, sr = gpu_run([pr], max_total_time_ns=TOP)
    rt, st = gpu_run([pr], max_total_time_ns=TOP, algo=B.ALGO_MERGE)
    with sr, st:
        rc, info = B.rannc_dp_solve_info(sr.h)
        assert info.level_kernel[3] == B.KERNEL_MERGE_RECOMPUTE
        for k in rr:
            assert np.array_equal(rr[k], rt[k]), k
        assert np.array_equal(sr.table(B.TABLE_V, 0), st.table(B.TABLE_V, 0))


def test_driver_equals_32_bit_tables():
    c = synth.form_stage_case(3, 404, 4, 8, 256, tight=3.0, tmax=2000, layered=True)
    args = (c["time_per_sample_ns"], c["act_bytes_per_sample"], c["param_bytes"], c["mem_capacity"])
    got = []
    for width, algo in ((B.NARROW_MAX_TOTAL_TIME, B.ALGO_MERGE), (TOP, B.ALGO_AUTO)):
        fs = B.FormStageSession(404, 4, 8, 256, max_total_time_ns=width, algo=algo)
        try:
            rc, out, se, rp = fs.run(*args)
            assert rc == B.OK and out.feasible
            vals = torch.empty((fs.Q, fs.max_D), dtype=torch.int64, device="cuda:0")
            assert B.rannc_dp_level_values(fs.h, torch.cuda.current_stream().cuda_stream, fs.max_D, vals) == B.OK
            torch.cuda.synchronize()
            got.append(((out.n, out.n_stages, out.n_microbatches, out.stage_time_ns, out.est_iter_ns), se, rp,
                        vals.cpu().numpy()))
        finally:
            fs.close()
    assert got[0][0] == got[1][0]
    for a, b in zip(got[0][1:], got[1][1:]):
        assert np.array_equal(a, b)
