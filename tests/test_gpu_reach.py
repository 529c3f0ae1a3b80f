"""Searches answered without their tables (rannc_dp_solve_to_host on a handle that leaves the kernels to the library)
against the oracle, where the kernel can go wrong: sizes at the edges of its loops and of what it takes, ties, chains
whose optimum leaves many cells open, too few stages, sums beyond its range.  And what such a call leaves behind: tables
made when they are asked for."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match, oracle_solve_many

pytestmark = pytest.mark.gpu


def _search(seed, N, D, S, kind="plain", share=1.6, scale=1):
    g = np.random.default_rng([seed, N, D, S])
    t, p, a = (g.integers(1, 1000, N).astype(np.int64) for _ in range(3))
    if kind == "equal":
        t[:], p[:], a[:] = 7, 11, 13
    if kind == "one long":
        t[N // 3] = 2 * t.sum()
    if kind == "zeros":
        t[:] = 0
    if kind == "transient":
        a *= 50
    M = int((p.sum() + a.sum()) / max(1, min(S, D, N)) * share) * scale
    return {"name": f"{kind}_{seed}_{N}_{D}_{S}", "time_ns": t, "param_bytes": p * scale, "act_bytes": a * scale, "n_devices": D,
            "max_stages": S, "n_microbatches": 8, "mem_capacity": M}


def _check(probs, **kw):
    with B.Session(synth.concat_batch(probs), **kw) as s:
        assert_results_match(probs, s.run(), oracle_results=oracle_solve_many(probs))


@pytest.mark.parametrize("N,D,S", [(1, 1, 1), (1, 64, 3), (2, 2, 2), (63, 33, 9), (64, 16, 8), (65, 17, 64), (192, 64, 12), (193, 8, 8), (576, 24, 6),
                                   (577, 3, 3), (1088, 5, 4), (1089, 40, 3), (4096, 2, 2), (4097, 2, 2)])
@pytest.mark.parametrize("share", [1.05, 1.6, 8.0])
def test_edges_of_the_sizes(N, D, S, share):
    _check([_search(1, N, D, S, share=share)])
    _check([_search(2, N, D, S, share=share)], max_total_time_ns=1 << 50)


@pytest.mark.parametrize("kind", ["equal", "one long", "zeros", "transient"])
@pytest.mark.parametrize("Q", [1, 64, 65, 513])   # each number of waves, with and without results in host memory
def test_open_plans_and_ties(kind, Q):
    g = np.random.default_rng(Q)
    probs = [_search(q, int(g.integers(2, 60)), int(g.integers(1, 65)), int(g.choice([1, 2, 3, 5, 64])), kind,
                     share=float(g.choice([0.8, 1.02, 1.3, 2.5]))) for q in range(Q)]
    _check(probs)


@pytest.mark.parametrize("N,D,S", [(40, 7, 6), (130, 17, 9), (251, 24, 15), (400, 64, 5), (1024, 40, 9), (2000, 33, 4)])
@pytest.mark.parametrize("grow", [1.0, 3.0])
@pytest.mark.parametrize("share", [1.01, 1.15, 1.4])
def test_many_open_cells_and_full_stages(N, D, S, grow, share):
    """Bytes that grow along the chain, so that a few blocks at its end take most stages (the bound leaves many cells, few of them
    reached), and stages nearly full, so that the stage limit binds; also as one of many searches."""
    pr = _search(9, N, D, S, share=share)
    weight = np.linspace(0.05, 1.0, N) ** grow
    pr["param_bytes"] = (pr["param_bytes"] * weight * 1000).astype(np.int64) + 1
    pr["mem_capacity"] = int((pr["param_bytes"].sum() + pr["act_bytes"].sum()) / min(S, D, N) * share)
    _check([pr])
    if N <= 251:
        _check([_search(q, 30, 5, 4) for q in range(66)] + [pr])


def test_beyond_the_exact_range_the_tables_decide():
    """Bytes of 2^46 and more in all, and times of 2^44 ns."""
    big = _search(3, 90, 12, 6, scale=1 << 31)
    assert big["param_bytes"].sum() > 1 << 46
    _check([big, _search(4, 80, 12, 6)])
    late = _search(5, 70, 20, 6)
    late["time_ns"] = late["time_ns"] << 29
    assert late["time_ns"].sum() > 1 << 44
    _check([late], max_total_time_ns=1 << 60)


def test_flagged_searches_among_others():
    probs = [_search(q, 50 + q, 9, 5) for q in range(4)]
    probs[1]["time_ns"][3] = -1
    probs[2]["param_bytes"][:] = 1 << 61
    probs[3]["time_ns"][:] = 1 << 30
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        assert list(res["status"]) == [0, B.PROBLEM_NEGATIVE_INPUT, B.PROBLEM_SUM_OVERFLOW, B.PROBLEM_TIME_TOO_LARGE]
        assert (res["opt"][1:] == B.INT64_MAX).all() and not res["n_stages"][1:].any() and (res["stage_end"][1:] == -1).all()
        assert_results_match(probs[:1], {k: v[:1] for k, v in res.items()})


def test_tables_are_made_from_what_the_call_was_given():
    """Inputs overwritten behind the call; the tables, level values and plans are still those of the searches it solved."""
    probs = [_search(q, 40 + 9 * q, (5, 16, 30, 64)[q % 4], 7) for q in range(6)]
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        for x in s.d_in:
            x.fill_(-1)
        d_v = torch.full((6, s.plan_stride), -5, dtype=torch.int64, device="cuda:0")
        assert B.rannc_dp_level_values(s.h, s.stream(), s.plan_stride, d_v) == B.OK
        s.d_se.fill_(-3)
        s.traceback()
        torch.cuda.synchronize()
        assert np.array_equal(s.d_se.cpu().numpy(), res["stage_end"])
        for q, pr in enumerate(probs):
            o = oracle.solve(pr, keep_tables=True)
            N, D, L = len(pr["time_ns"]), pr["n_devices"], o["n_levels"]
            assert np.array_equal(s.table(B.TABLE_V, q), o["V"])
            assert np.array_equal(d_v.cpu().numpy()[q, :L], o["V"][1:L + 1, N, D])


def test_plan_recovery_recorded_behind_the_call():
    probs = [_search(q, 60, 12, 6) for q in range(3)]
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            assert B.rannc_dp_traceback(s.h, torch.cuda.current_stream().cuda_stream, s.plan_stride, s.d_se, s.d_rp) == B.OK
        for _ in range(3):
            s.d_se.fill_(-3)
            s.d_rp.fill_(-3)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(s.d_se.cpu().numpy(), res["stage_end"]) and np.array_equal(s.d_rp.cpu().numpy(), res["replicas"])
        assert np.array_equal(s.table(B.TABLE_V, 1), oracle.solve(probs[1], keep_tables=True)["V"])


@pytest.mark.parametrize("form", ["", "s"])
def test_a_recorded_recovery_follows_later_calls(form):
    """Plans and level values recorded behind one call and replayed behind later ones of the same shapes: each replay is of the call
    in front of it."""
    def batch(seed):
        probs = [_search(seed + q, 60, 12, 6) for q in range(3)]
        for pr in probs if form else []:
            pr["time_bwd_ns"] = pr["time_ns"][::-1].copy()
        return probs
    with B.Session(synth.concat_batch(batch(0))) as s:
        s.run()
        d_v = torch.zeros((3, s.plan_stride), dtype=torch.int64, device="cuda:0")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            st = torch.cuda.current_stream().cuda_stream
            assert B.rannc_dp_traceback(s.h, st, s.plan_stride, s.d_se, s.d_rp) == B.OK
            assert B.rannc_dp_level_values(s.h, st, s.plan_stride, d_v) == B.OK
        for seed in (0, 10, 20):
            probs = batch(seed)
            b = synth.concat_batch(probs)
            for x, key in zip(s.d_in + [s.d_bwd] * bool(form), ("time_ns", "param_bytes", "act_bytes", "time_bwd_ns")):
                x.copy_(torch.from_numpy(np.ascontiguousarray(b[key], dtype=np.int64)))
            s.hb.keep[4][:] = b["mem_capacity"]
            res = s.run()
            assert_results_match(probs, res)
            for x in (s.d_se, s.d_rp):
                x.fill_(-3)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(s.d_se.cpu().numpy(), res["stage_end"]) and np.array_equal(s.d_rp.cpu().numpy(), res["replicas"])
            for q, pr in enumerate(probs):
                o = oracle.solve(pr, keep_tables=True)
                assert np.array_equal(d_v.cpu().numpy()[q, :o["n_levels"]], o["V"][1:o["n_levels"] + 1, 60, 12])


def test_a_recorded_solve_behind_other_calls():
    """A whole solve recorded and replayed behind a call of its own: the recovery behind the replay is of the replay's inputs."""
    first, second = [_search(1, 60, 12, 6)], [_search(2, 60, 12, 6)]
    want = oracle.solve(first[0])
    with B.Session(synth.concat_batch(first)) as s:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            st = torch.cuda.current_stream().cuda_stream
            assert B.rannc_dp_solve(s.h, s.hb, st, s.d_opt, s.d_ns, s.d_est, s.d_status) == B.OK
        b = synth.concat_batch(second)
        others = [torch.from_numpy(np.ascontiguousarray(b[k], dtype=np.int64)).to("cuda:0") for k in ("time_ns", "param_bytes", "act_bytes")]
        hb = B.HostBatch(b["n_blocks"], b["n_devices"], b["max_stages"], b["n_microbatches"], b["mem_capacity"], b["block_offset"], *others)
        out = np.zeros(s._out_dev.numel(), np.uint8)
        for _ in range(2):
            assert B.rannc_dp_solve_to_host(s.h, hb, s.stream(), s.plan_stride, s._out_dev, out, out.nbytes) == B.OK
            assert int(out[:8].view(np.int64)[0]) == oracle.solve(second[0])["opt"]
            graph.replay()
            s.traceback()
            torch.cuda.synchronize()
            assert int(s.d_opt.item()) == want["opt"]
            assert np.array_equal(s.d_se.cpu().numpy()[0][:want["n_levels"]], want["stage_end"])


def long_work(stream):
    """Work of tens of milliseconds on the stream; the event behind it has not happened behind a call that does not wait."""
    with torch.cuda.stream(stream):
        torch.cuda._sleep(200_000_000)
        return stream.record_event()


def test_recovery_behind_the_call_does_not_wait():
    """Plan recovery, level values and tables behind a call answered without tables only enqueue, as behind a solve; work on another
    stream behind them waits for the tables on the device."""
    probs = [_search(q, 60, (12, 60)[q % 2], 6) for q in range(4)]
    with B.Session(synth.concat_batch(probs)) as s:
        one, other = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(one):
            res = s.run()
        s.d_se.fill_(-3)
        s.d_rp.fill_(-3)
        d_v = torch.full((4, s.plan_stride), -5, dtype=torch.int64, device="cuda:0")
        torch.cuda.synchronize()
        done = long_work(one)
        assert B.rannc_dp_traceback(s.h, one.cuda_stream, s.plan_stride, s.d_se, s.d_rp) == B.OK
        assert B.rannc_dp_level_values(s.h, other.cuda_stream, s.plan_stride, d_v) == B.OK
        assert not done.query()
        other.synchronize()
        for q, pr in enumerate(probs):
            o = oracle.solve(pr, keep_tables=True)
            N, D, L = len(pr["time_ns"]), pr["n_devices"], o["n_levels"]
            assert np.array_equal(d_v.cpu().numpy()[q, :L], o["V"][1:L + 1, N, D])
        torch.cuda.synchronize()
        assert np.array_equal(s.d_se.cpu().numpy(), res["stage_end"]) and np.array_equal(s.d_rp.cpu().numpy(), res["replicas"])


def test_a_program_that_reads_the_tables_pays_for_one_search():
    """Where the tables were asked for behind a call, the next one makes its own; where they were not, it is answered without."""
    probs = [_search(3, 60, 12, 6)]
    want = oracle.solve(probs[0], keep_tables=True)
    with B.Session(synth.concat_batch(probs)) as s:
        assert B.rannc_dp_answered_without_tables(s.h) == B.BAD_STATE
        for ask, direct in ((False, 1), (True, 1), (True, 0), (False, 0), (True, 1), (False, 0), (False, 1), (False, 1)):
            assert_results_match(probs, s.run(), oracle_results=[want])
            assert B.rannc_dp_answered_without_tables(s.h) == direct
            if ask:
                assert np.array_equal(s.table(B.TABLE_V, 0), want["V"])
                assert B.rannc_dp_answered_without_tables(s.h) == direct
        s.solve()
        s.traceback()
        assert B.rannc_dp_answered_without_tables(s.h) == 0
        s.run()     # (behind a solve that a program reads on the device nothing was put off)
        assert B.rannc_dp_answered_without_tables(s.h) == 1


def test_the_kernels_reported_are_those_that_make_the_tables():
    """A workspace that holds the batch as one group, or class by class beside the copies of its inputs, but not as a group beside them."""
    probs = [_search(q, 40, D, 6) for q, D in enumerate((8, 8, 8, 64))]
    with B.Session(synth.concat_batch(probs)) as s:
        copies = (5 * 8 * 160 + 255) // 256 * 256 + 256
        rc, h = B.rannc_dp_create(s.limits, s.ws, s.ws_bytes - copies)
        assert rc == B.OK
        try:
            out = np.zeros(s._out_dev.numel(), np.uint8)
            assert B.rannc_dp_solve_to_host(h, s.hb, s.stream(), s.plan_stride, s._out_dev, out, out.nbytes) == B.OK
            assert B.rannc_dp_answered_without_tables(h) == 4
            rc, before = B.rannc_dp_solve_info(h)
            assert rc == B.OK
            d_v = torch.zeros((4, s.plan_stride), dtype=torch.int64, device="cuda:0")
            assert B.rannc_dp_level_values(h, s.stream(), s.plan_stride, d_v) == B.OK
            rc, after = B.rannc_dp_solve_info(h)
            assert rc == B.OK and list(before.n_problems) == list(after.n_problems) == [3, 0, 0, 1]
            assert list(before.level_kernel) == list(after.level_kernel)
            torch.cuda.synchronize()
            for q, pr in enumerate(probs):
                o = oracle.solve(pr, keep_tables=True)
                assert np.array_equal(d_v.cpu().numpy()[q, :o["n_levels"]], o["V"][1:o["n_levels"] + 1, 40, pr["n_devices"]])
        finally:
            torch.cuda.synchronize()
            B.rannc_dp_destroy(h)


@pytest.mark.parametrize("N,D,S", [(51, 64, 20), (185, 17, 9), (215, 16, 8)])
def test_sizes_whose_lds_lies_about_64_kib(N, D, S):
    _check([_search(1, N, D, S, share=1.3)])


@pytest.mark.parametrize("Q,comm", [(2, False), (8, False), (64, False), (65, False), (200, False), (2, True), (8, True), (64, True)])
def test_open_searches_are_solved_by_themselves(Q, comm):
    """Searches whose sums lie beyond the kernel's range among others, at both ends and in between: their tables alone are made, every
    result stands in its place on the host and on the device, and tables asked for behind the call are the whole batch's."""
    probs = [_search(q, 161 if comm else 30 + q % 40, (4, 5, 8)[q % 3], 5) for q in range(Q)]
    odd = sorted({0, Q // 2, Q - 1} if Q > 2 else {1})
    for q in odd:
        probs[q] = _search(1000 + q, 161 if comm else 50, 7, 6, scale=1 << 33)
    for pr in probs if comm else []:
        g = np.random.default_rng(pr["n_devices"])
        pr["cut_bytes"], pr["bandwidth_bytes_per_us"] = g.integers(0, 300, len(pr["time_ns"])), 1000
    want = oracle_solve_many(probs)
    with B.Session(synth.concat_batch(probs)) as s:
        for again in range(2):
            s._out_dev.fill_(77)
            res = s.run()
            assert B.rannc_dp_answered_without_tables(s.h) == Q - len(odd)
            assert_results_match(probs, res, oracle_results=want)
            if Q > 64:   # (few searches write their results to the host alone)
                assert np.array_equal(s.d_opt.cpu().numpy(), res["opt"]) and np.array_equal(s.d_se.cpu().numpy(), res["stage_end"])
        for q in (odd[0], (odd[0] + 1) % Q):
            assert np.array_equal(s.table(B.TABLE_V, q), oracle.solve(probs[q], keep_tables=True)["V"])
        s.d_se.fill_(-3)
        s.traceback()
        torch.cuda.synchronize()
        assert np.array_equal(s.d_se.cpu().numpy(), res["stage_end"])


@pytest.mark.parametrize("N,D,S,kind,share", [(175, 11, 5, "plain", 0.78), (22, 15, 7, "plain", 0.82), (668, 33, 33, "one long", 1.3),
                                              (1400, 23, 23, "one long", 1.3), (1024, 64, 9, "plain", 0.65)])
def test_what_is_left_to_the_tables(N, D, S, kind, share):
    """Stages that hardly hold the bytes, and a block longer than the others: as soon as it shows that the tables are
    quicker the kernel leaves the search to them, alone and among others; with room to spare it does not."""
    pr, others = _search(7, N, D, S, kind, share), [_search(q, 40, 8, 5, share=3.0) for q in range(70)]
    want = [oracle.solve(pr)] + oracle_solve_many(others)
    for probs, least, most in (([pr], 0, 0), ([pr] + others, 70, 71), ([_search(7, N, D, S, share=6.0)], 1, 1)):
        with B.Session(synth.concat_batch(probs)) as s:
            res = s.run()
            assert least <= B.rannc_dp_answered_without_tables(s.h) <= most
            if probs[0] is pr:
                assert_results_match(probs, res, oracle_results=want)


@pytest.mark.parametrize("kind", ["plain", "equal", "one long", "transient"])
@pytest.mark.parametrize("Q", [1, 64, 65, 512])
def test_usual_searches_are_answered_by_the_kernel(kind, Q):
    """Results are the same where the tables take over: here that they do not."""
    g = np.random.default_rng([Q, 3])
    probs = [_search(q, int(g.integers(2, 60)), int(g.integers(1, 65)), int(g.choice([1, 2, 3, 5, 64])), kind if q % 2 else "plain", share=2.5)
             for q in range(Q)]
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        assert B.rannc_dp_answered_without_tables(s.h) >= Q - Q // 50   # (of equal blocks a few leave more cells than there is room for)
        assert_results_match(probs, res, oracle_results=oracle_solve_many(probs))


@pytest.mark.parametrize("N,D,S,n", [(1, 1, 1, 1), (64, 16, 8, 1), (192, 64, 12, 1), (577, 3, 3, 1), (1089, 40, 3, 1), (4096, 2, 2, 1), (4097, 2, 2, 0)])
def test_sizes_that_the_kernel_takes(N, D, S, n):
    for algo, want in ((B.ALGO_AUTO, n), (B.ALGO_MERGE, 0)):
        with B.Session(synth.concat_batch([_search(1, N, D, S)]), algo=algo) as s:
            s.run()
            assert B.rannc_dp_answered_without_tables(s.h) == want
