"""The launches that list the stages that fit: setup, tables and level 1 of searches of up to 1024 blocks
as one kernel, the level kernel's passes of 64 listed stages, the one-launch kernel with the plans
recovered in it, and the split objective's levels that unpack the level before.  Sizes at the edges of
chunks, workgroups and lists, bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match, assert_tables_match, gpu_run

pytestmark = pytest.mark.gpu

NARROW, WIDE = B.NARROW_MAX_TOTAL_TIME, B.WIDE_RECOMPUTE_MAX_TOTAL_TIME


def _scaled(pr, width):
    """64-bit handles get stage times beyond 32 bits, most of them one above a multiple of a replica count."""
    return pr if width == NARROW else dict(pr, time_ns=pr["time_ns"] * (840 << 10) + 1)


@pytest.mark.parametrize("width", [NARROW, WIDE])
@pytest.mark.parametrize("N", [1, 62, 63, 64, 65, 128, 129, 255, 256, 257, 1023, 1024, 1025])
def test_setup_and_tables(N, width):
    """One search (workgroups of 1024) and nine (workgroups of 256) of the same length and a shorter one, with
    memory for single blocks only, with a block that fits nowhere, and with memory that never binds; 1025 blocks
    take the separate kernels."""
    def case(k, tight):
        return _scaled(synth.random_small(31 * N + k, max(1, N - (k == 4)), 8, 3, tight=tight, tmax=9), width)
    few = [case(0, 2.0)]
    many = [case(k, (1.01, 2.0, 60.0)[k % 3]) for k in range(9)]
    n = many[3]["time_ns"].shape[0]
    many[3] = dict(many[3], param_bytes=many[3]["param_bytes"].copy())
    many[3]["param_bytes"][n // 2] = 1 << 45  # fits nowhere
    for probs in (few, many):
        res, sess = gpu_run(probs, max_total_time_ns=width, one_launch_small=1)
        with sess:
            assert_results_match(probs, res)
            for q in (0, len(probs) // 2):
                assert_tables_match(probs[q], sess, q, args=False)


@pytest.mark.parametrize("width", [NARROW, WIDE])
@pytest.mark.parametrize("N,D,S", [(64, 8, 8), (100, 64, 64), (130, 32, 32), (700, 16, 16)])
def test_passes_of_many_rows(N, D, S, width):
    """Equal blocks and memory for 1, 2, 3 and 40 of them on one device: a pass of 64 stages holds from one row
    to far more rows than are kept near."""
    one = synth.random_small(5, N, D, S, tight=1.0, tmax=50)
    block = np.full(N, 1 << 30, dtype=np.int64)
    probs = [_scaled(dict(one, param_bytes=block, act_bytes=block // 64, mem_capacity=int(k * (1 << 30) * 1.1)), width)
             for k in (1, 2, 3, 40)]
    res, sess = gpu_run(probs, max_total_time_ns=width, one_launch_small=1, algo=B.ALGO_RECOMPUTE)
    with sess:
        assert_results_match(probs, res)
        for q in range(len(probs)):
            assert_tables_match(probs[q], sess, q, args=False)


@pytest.mark.parametrize("width", [NARROW, WIDE])
@pytest.mark.parametrize("comm", [False, True])
@pytest.mark.parametrize("N", [1, 2, 17, 32, 33, 62, 63, 64, 65, 66, 127, 128])
def test_one_launch_with_plans(N, comm, width):
    """Several searches of one class, their plans recovered in the launch: few levels (all of them held in LDS)
    and as many as devices, a flagged search among them, and a call for each of them alone."""
    for D, S in ((8, 3), (8, 8), (32, 2), (32, 32)):
        probs = [_scaled(synth.random_small(100 * N + D + S + k, N, D, S, tight=(1.2, 3.0, 50.0)[k], tmax=9), width)
                 for k in range(3)]
        if comm:
            probs = [synth.with_cut_bytes(p, 17 + k, 1 << 30) for k, p in enumerate(probs)]
        bad = dict(probs[1], act_bytes=probs[1]["act_bytes"].copy())
        bad["act_bytes"][N // 2] = -1
        res, sess = gpu_run(probs + [bad], max_total_time_ns=width, one_launch_small=2)
        with sess:
            assert list(res["status"]) == [B.PROBLEM_OK] * 3 + [B.PROBLEM_NEGATIVE_INPUT]
            assert (res["stage_end"][3] == -1).all()
            assert_results_match(probs, {k: v[:3] for k, v in res.items()})
        alone, sess = gpu_run(probs[:1], max_total_time_ns=width, one_launch_small=2)
        with sess:
            assert_results_match(probs[:1], alone)


@pytest.mark.parametrize("width", [NARROW, 1 << 50])
@pytest.mark.parametrize("N", [15, 16, 17, 100])
def test_split_levels_of_mixed_stage_counts(N, width):
    """Searches that end at level 1, 2, 3, 4 and 9 in one launch: each level's winners are unpacked in the next
    one's launch for searches that end there as well."""
    probs = [synth.with_backward_times(synth.random_small(9 * N + S, N, 9, S, tight=1.5 + S % 2 * 20, tmax=9), 3, tmax=9)
             for S in (1, 2, 3, 4, 9)]
    res, sess = gpu_run(probs, max_total_time_ns=width)
    with sess:
        assert_results_match(probs, res)
        for q in range(len(probs)):
            assert_tables_match(probs[q], sess, q)
