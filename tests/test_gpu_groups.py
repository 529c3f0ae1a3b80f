"""Batches of few searches: as one group padded to the widest device-count class, or class by class where
the narrower searches hold too many rows (or the workspace too little).  The number of level launches
tells which of the two ran."""
import numpy as np
import pytest
import torch

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match

pytestmark = pytest.mark.gpu
NARROW, WIDE = B.NARROW_MAX_TOTAL_TIME, B.WIDE_RECOMPUTE_MAX_TOTAL_TIME


def _batch(shapes, split):
    probs = [synth.random_small(40 + q, N, D, 5 if q + 1 < len(shapes) else 7, tight=2.0) for q, (N, D) in enumerate(shapes)]
    return [synth.with_backward_times(p, 3, tmax=50) for p in probs] if split else probs


def _level_launches(s):
    assert B.rannc_dp_set_timing(s.h, True) == B.OK
    s.run()
    return B.rannc_dp_get_timing(s.h)[2]


# rows of a search: 1024 blocks 8704, 160 blocks 352, 64 blocks 64, one block 1
@pytest.mark.parametrize("shapes,split,bound,group", [
    ([(1024, 8)] * 6 + [(300, 64)], False, NARROW, False),
    ([(160, 8)] * 16 + [(160, 64)], False, NARROW, True),                # 5632 rows, the last that fit
    ([(160, 8)] * 16 + [(1, 8), (160, 64)], False, NARROW, False),
    ([(160, 8)] * 15 + [(160, 16), (1, 16), (160, 64)], False, NARROW, True),   # a third class
    ([(160, 16)] * 29 + [(32, 16), (160, 32)], False, NARROW, True),     # 10240 rows
    ([(160, 16)] * 29 + [(33, 16), (160, 32)], False, NARROW, False),
    ([(64, 8)] * 22 + [(160, 64)], False, WIDE, True),                   # 1408 rows
    ([(64, 8)] * 22 + [(1, 8), (160, 64)], False, WIDE, False),
    ([(64, 16)] * 28 + [(64, 32)], True, NARROW, True),                  # 1792 rows
    ([(64, 16)] * 28 + [(1, 16), (64, 32)], True, NARROW, False),
])
def test_a_group_only_while_the_narrower_searches_are_small(shapes, split, bound, group):
    probs = _batch(shapes, split)
    with B.Session(synth.concat_batch(probs), max_total_time_ns=bound, one_launch_small=1) as s:
        assert_results_match(probs, s.run())
        # the levels of the widest search, and apart from them those of every narrower class
        assert _level_launches(s) == 6 + (0 if group else 4)


def test_a_group_that_does_not_fit_the_workspace_runs_class_by_class():
    probs = _batch([(100, 8)] * 30 + [(20, 64)], False)     # 4920 rows: a group where there is room
    with B.Session(synth.concat_batch(probs), one_launch_small=1) as s:
        want = s.run()
        assert_results_match(probs, want)
        assert _level_launches(s) == 6

        def alone(n, *which):  # workspace of n copies of a search
            b = synth.concat_batch([probs[q] for q in which for _ in range(n)])
            z = np.zeros(1, dtype=np.int64)  # (the query looks at the sizes only)
            return B.rannc_dp_workspace_bytes_for(s.limits, B.HostBatch(
                b["n_blocks"], b["n_devices"], b["max_stages"], b["n_microbatches"], b["mem_capacity"],
                b["block_offset"], z, z, z))
        header = 2 * alone(1, 0) - alone(2, 0)
        nbytes = header + 30 * (alone(1, 0) - header) + (alone(1, 30) - header)
        assert nbytes < s.ws_bytes
        ws = torch.empty(nbytes, dtype=torch.uint8, device=s.dev)
        rc, other = B.rannc_dp_create(s.limits, ws, nbytes)
        assert rc == B.OK
        try:
            s._out_host.zero_()
            rc = B.rannc_dp_solve_to_host(other, s.hb, s.stream(), s.plan_stride, s._out_dev, s._out_host, s._out_host.numel())
            assert rc == B.OK
            for key, v in zip(("opt", "est_iter_ns", "n_stages", "status", "stage_end", "replicas"), s._h_views):
                assert np.array_equal(v, want[key]), key
            assert B.rannc_dp_set_timing(other, True) == B.OK
            assert B.rannc_dp_solve(other, s.hb, s.stream(), s.d_opt, s.d_ns, s.d_est, s.d_status) == B.OK
            assert B.rannc_dp_get_timing(other)[2] == 6 + 4
        finally:
            torch.cuda.synchronize()
            B.rannc_dp_destroy(other)


@pytest.mark.parametrize("narrow", [3, 20])      # one group; class by class on streams of the handle
def test_recorded_into_a_graph_and_replayed(narrow):
    probs = _batch([(160, 8)] * narrow + [(160, 64)], False)
    with B.Session(synth.concat_batch(probs)) as s:
        want = s.run()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            s.solve()
            s.traceback()
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            s.solve()
            s.traceback()
        for _ in range(4):
            s.d_opt.fill_(-7)
            s.d_se.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(s.d_opt.cpu().numpy(), want["opt"])
            assert np.array_equal(s.d_se.cpu().numpy(), want["stage_end"])
        for _ in range(3):
            assert_results_match(probs, s.run())
