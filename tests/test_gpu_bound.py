"""Searches with send times, and with forward and backward maxima apart, answered without their tables
(rannc_dp_solve_to_host) against the oracle, where the kernel can go wrong: sizes at the edges of its loops and of what it takes, ties,
send times from none to many blocks long, chains that memory cuts and chains that it does not, too few stages, and more cells
than it holds.  And what such a call leaves behind: tables made when they are asked for."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match, oracle_solve_many

pytestmark = pytest.mark.gpu


def _search(seed, N, D, S, form, kind="plain", share=1.6, cut=1000, top=1000):
    """form: "c" send times, "s" maxima apart, "cs" both; cut: longest send time in ns, top: longest block."""
    g = np.random.default_rng([seed, N, D, S])
    t, p, a = (g.integers(1, 1000, N).astype(np.int64) for _ in range(3))
    t = g.integers(1, top + 1, N).astype(np.int64)
    b = g.integers(0, 2 * top + 1, N).astype(np.int64)
    o = g.integers(0, cut + 1, N).astype(np.int64)
    if kind == "equal":
        t[:], p[:], a[:], b[:], o[:] = 7, 11, 13, 5, min(cut, 3)
    if kind == "small":     # many equal values
        t, b, o = t % 4, b % 3, o % 3
    if kind == "one long":
        t[N // 3] = 2 * t.sum()
    if kind == "zeros":
        t[:], b[:] = 0, 0
    if kind == "opposed":   # long forward where backward is short
        b = top + 1 - t
    M = int((p.sum() + a.sum()) / max(1, min(S, D, N)) * share)
    pr = {"name": f"{form}_{kind}_{seed}_{N}_{D}_{S}", "time_ns": t, "param_bytes": p, "act_bytes": a, "n_devices": D, "max_stages": S,
          "n_microbatches": 8, "mem_capacity": M}
    if "s" in form:
        pr["time_bwd_ns"] = b
    if "c" in form:
        pr["cut_bytes"], pr["bandwidth_bytes_per_us"] = o, 1000
    return pr


def _check(probs, **kw):
    with B.Session(synth.concat_batch(probs), **kw) as s:
        assert_results_match(probs, s.run(), oracle_results=oracle_solve_many(probs))


@pytest.mark.parametrize("form", ["c", "s", "cs"])
@pytest.mark.parametrize("N,D,S", [(1, 1, 1), (1, 64, 3), (2, 2, 2), (17, 8, 8), (63, 33, 9), (64, 16, 8), (65, 17, 64), (193, 8, 8), (300, 64, 12),
                                   (577, 3, 3), (1024, 5, 4), (1025, 4, 3)])
@pytest.mark.parametrize("share", [1.05, 1.6, 8.0])
def test_edges_of_the_sizes(form, N, D, S, share):
    if N > 300 and share == 1.6:
        D = min(D, 4)
    _check([_search(1, N, D, S, form, share=share)])
    _check([_search(2, N, D, S, form, share=share, cut=20000)], max_total_time_ns=1 << 50)


@pytest.mark.parametrize("form", ["c", "s", "cs"])
@pytest.mark.parametrize("kind", ["plain", "equal", "small", "one long", "zeros", "opposed"])
@pytest.mark.parametrize("Q", [1, 64, 65])
def test_open_plans_and_ties(form, kind, Q):
    g = np.random.default_rng([Q, len(form), len(kind)])
    for _ in range(12 if Q == 1 else 1):
        probs = [_search(int(g.integers(1 << 30)), int(g.integers(2, 60)), int(g.integers(1, 65)), int(g.choice([1, 2, 3, 5, 64])), form, kind,
                         share=float(g.choice([0.8, 1.02, 1.3, 2.5])), cut=int(g.choice([0, 3, 300, 50000]))) for q in range(Q)]
        _check(probs)


@pytest.mark.parametrize("form", ["c", "s", "cs"])
def test_searches_of_more_cells_than_the_kernel_holds(form):
    """Send times and blocks so uneven that the bound leaves nearly every cell; and two searches that it settles beside one."""
    hard = _search(5, 220, 40, 30, form, "opposed", share=2.0, cut=10**6, top=20)
    _check([hard])
    _check([_search(6, 50, 9, 5, form), hard, _search(7, 90, 33, 7, form)])


@pytest.mark.parametrize("form", ["c", "s", "cs"])
def test_flagged_searches_among_others(form):
    probs = [_search(q, 50 + q, 9, 5, form) for q in range(5)]
    probs[1]["time_ns"][3] = -1
    probs[2]["param_bytes"][:] = 1 << 61
    probs[3]["time_ns"][:] = 1 << 30
    want = [0, B.PROBLEM_NEGATIVE_INPUT, B.PROBLEM_SUM_OVERFLOW, B.PROBLEM_TIME_TOO_LARGE, 0]
    if "c" in form:
        probs[4]["cut_bytes"][:] = 1 << 60
        want[4] = B.PROBLEM_SUM_OVERFLOW
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        assert list(res["status"]) == want
        assert_results_match(probs[:1], {k: v[:1] for k, v in res.items()})


@pytest.mark.parametrize("form", ["c", "s", "cs"])
def test_tables_are_made_from_what_the_call_was_given(form):
    probs = [_search(q, 40 + 9 * q, (5, 16, 30, 64)[q % 4], 7, form) for q in range(4)]
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        for x in s.d_in:
            x.fill_(-1)
        d_v = torch.full((4, s.plan_stride), -5, dtype=torch.int64, device="cuda:0")
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


def _in_line(g, form):
    """Blocks, devices, stages of a search that the kernel is asked for: with send times few devices or stages, and with one
    objective chains that are not one launch with tables."""
    while True:
        D, S = int(g.integers(1, 33)), int(g.choice([1, 2, 3, 5, 8]))
        if "c" not in form or D * min(S, D) <= 64:
            return (int(g.integers(161, 300)) if form == "c" else int(g.integers(2, 60))), D, S


@pytest.mark.parametrize("form", ["c", "s", "cs"])
@pytest.mark.parametrize("kind", ["plain", "equal", "small", "one long", "opposed"])
@pytest.mark.parametrize("Q", [1, 7, 64])
def test_searches_that_the_kernel_answers(form, kind, Q):
    """With room to spare every one is answered without tables; nearly full, with long send times, and without a plan results agree
    whichever way they come."""
    g = np.random.default_rng([Q, len(kind), len(form)])
    for share, cut, settled in ((2.5, 3, True), (2.5, 300, True), (6.0, 300, True), (1.02, 50000, False), (0.8, 300, False)):
        probs = [_search(int(g.integers(1 << 30)), *_in_line(g, form), form, kind, share=share, cut=cut) for q in range(Q)]
        with B.Session(synth.concat_batch(probs), max_total_time_ns=1 << 42) as s:
            res = s.run()
            if settled:
                assert B.rannc_dp_answered_without_tables(s.h) >= Q - Q // 16   # (ties can leave more cells than there is room for)
            assert_results_match(probs, res, oracle_results=oracle_solve_many(probs))


@pytest.mark.parametrize("form,N,D,S,Q,n", [("c", 160, 4, 3, 1, 0), ("c", 161, 4, 3, 1, 1), ("c", 300, 13, 5, 1, 0), ("c", 300, 32, 2, 1, 1), ("c", 200, 4, 3, 65, 0),
                                            ("c", 1024, 4, 3, 1, 1), ("c", 1025, 4, 3, 1, 0), ("cs", 20, 8, 8, 1, 1), ("cs", 20, 9, 8, 1, 0),
                                            ("s", 20, 40, 20, 64, 64), ("s", 20, 4, 4, 65, 0), ("s", 1025, 3, 3, 1, 0)])
def test_which_searches_the_kernel_is_asked_for(form, N, D, S, Q, n):
    probs = [_search(q, N, D, S, form, share=3.0) for q in range(Q)]
    with B.Session(synth.concat_batch(probs), max_total_time_ns=1 << 42) as s:
        res = s.run()
        assert B.rannc_dp_answered_without_tables(s.h) == n
        if N < 1000:
            assert_results_match(probs[:2], {k: v[:2] for k, v in res.items()}, oracle_results=oracle_solve_many(probs[:2]))


@pytest.mark.parametrize("form", ["c", "cs"])
def test_flags_and_tables_of_searches_the_kernel_answers(form):
    """Inputs that are refused, and tables made from the saved bytes per cut and bandwidths, inside of what the kernel takes."""
    probs = [_search(q, 170 + 9 * q, (3, 8, 20, 5)[q % 4], (5, 8, 3, 5)[q % 4], form, share=3.0) for q in range(4)]
    for q, pr in enumerate(probs):
        pr["bandwidth_bytes_per_us"] = 500 + 300 * q
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        assert B.rannc_dp_answered_without_tables(s.h) == 4
        assert_results_match(probs, res, oracle_results=oracle_solve_many(probs))
        for x in s.d_in + [s.d_cut] + ([s.d_bwd] if "s" in form else []):
            x.fill_(-1)
        s.d_se.fill_(-3)
        s.traceback()
        torch.cuda.synchronize()
        assert np.array_equal(s.d_se.cpu().numpy(), res["stage_end"])
        for q, pr in enumerate(probs):
            assert np.array_equal(s.table(B.TABLE_V, q), oracle.solve(pr, keep_tables=True)["V"])
    probs[0]["cut_bytes"][-2] = 1 << 60
    probs[1]["cut_bytes"][0] = -1
    probs[2]["time_ns"][:] = 1 << 30
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        assert B.rannc_dp_answered_without_tables(s.h) == 4
        assert list(res["status"]) == [B.PROBLEM_SUM_OVERFLOW, B.PROBLEM_NEGATIVE_INPUT, B.PROBLEM_TIME_TOO_LARGE, B.PROBLEM_OK]
        assert_results_match(probs[3:], {k: v[3:] for k, v in res.items()})
