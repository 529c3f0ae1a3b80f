"""The launches that list the stages that fit: setup, tables and level 1 of searches of up to 1024 blocks
as one kernel, the level kernel's passes of 64 listed stages, the one-launch kernel with the plans
recovered in it, and the split objective's levels that unpack the level before.  Sizes at the edges of
chunks, workgroups and lists, bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
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


@pytest.mark.parametrize("N,huge", [(1025, False), (1100, True), (2048, False), (2049, False), (4096, False), (4097, False),
                                    (4098, True)])
def test_lists_of_long_chains(N, huge):
    """Searches of more than 1024 blocks: the ends searched in LDS (up to 4096 blocks), out of memory, and with bytes
    whose sums per device would wrap.  Memory for half the chain, for some forty blocks, the same with blocks that fit
    nowhere (the first one of a chunk, and all of another), memory that never binds, short chains and a flagged
    search beside them."""
    def case(k, D, tight, S=3):
        return synth.random_small(17 * N + k, N, D, S, tight=tight, tmax=9)
    short = [synth.random_small(3, n, 6, 3, tight=2.0, tmax=9) for n in (1, 65)]
    probs = [case(0, 4, 1.5), case(1, 3, 1.0), case(2, 8, 60.0), case(4, 8, 1.0, 8), *short, case(3, 5, 2.0)]
    for few in (probs[1], probs[3]):
        few["mem_capacity"] = int((few["param_bytes"].mean() + few["act_bytes"].mean()) * 40)
    few = probs[1]
    few["param_bytes"][[128, 129, 700, 1023]] = few["mem_capacity"] + 1
    few["param_bytes"][320:384] = few["mem_capacity"] + 1
    if huge:
        for pr in probs:
            up = (1 << 57) // int(pr["param_bytes"].sum() + pr["act_bytes"].sum())
            for key in ("param_bytes", "act_bytes", "mem_capacity"):
                pr[key] = pr[key] * up
    probs[6]["act_bytes"][N // 3] = -1
    res, sess = gpu_run(probs)
    with sess:
        rc, info = B.rannc_dp_solve_info(sess.h)
        assert rc == B.OK and info.level_kernel[0] == B.KERNEL_MERGE_RECOMPUTE
        assert list(res["status"]) == [B.PROBLEM_OK] * 6 + [B.PROBLEM_NEGATIVE_INPUT]
        assert_results_match(probs[:6], {k: v[:6] for k, v in res.items()})
        for q in range(6):
            o = oracle.solve(probs[q], keep_tables=True)
            assert np.array_equal(sess.table(B.TABLE_V, q), o["V"]), q
            assert np.array_equal(sess.table(B.TABLE_FIT, q), o["fit"]), q
        if N < 1200:
            assert_tables_match(probs[0], sess, 0, args=False)


@pytest.mark.parametrize("Q,N", [(2, 512), (2, 513), (16, 513), (17, 513), (64, 256), (65, 256), (65, 257)])
def test_tables_of_several_searches(Q, N):
    """Sums and tables as one launch or two: either side of the lines, with send times."""
    distinct = [synth.with_cut_bytes(synth.random_small(7 * N + k, N - k, (6, 8, 7)[k], 3, tight=(1.5, 3.0, 40.0)[k], tmax=99), k, 1000)
                for k in range(3)]
    probs = [distinct[q % 3] for q in range(Q)]
    res, sess = gpu_run(probs, one_launch_small=1)
    with sess:
        rc, info = B.rannc_dp_solve_info(sess.h)
        assert rc == B.OK and info.level_kernel[0] == B.KERNEL_MERGE_TABLE
        want = [oracle.solve(pr) for pr in distinct]
        assert_results_match(probs, res, oracle_results=[want[q % 3] for q in range(Q)])
        for q in (1, Q - 1):
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
