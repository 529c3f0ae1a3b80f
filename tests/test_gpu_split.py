"""GPU parity of Algorithm 1 as printed (forward and backward maxima carried separately, handles
with RANNC_DP_FLAG_SPLIT_OBJECTIVE) against the CPU oracle's run of the same steps: both stage-time
tables, values, the carried maxima, the kept candidates and the plans.  Integers: bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import INF, assert_results_match, assert_tables_match, gpu_run

pytestmark = pytest.mark.gpu

WIDTHS = [B.NARROW_MAX_TOTAL_TIME, 1 << 50]
SHAPES = [(1, 1, 1), (1, 7, 3), (9, 1, 4), (5, 2, 5), (16, 4, 4), (33, 5, 5), (63, 8, 8), (64, 9, 6),
          (65, 12, 7), (100, 17, 9), (129, 24, 6), (130, 33, 5), (70, 63, 10), (96, 64, 12), (72, 64, 64)]


def _case(seed, N, D, S, tight, tmax, comm):
    pr = synth.with_backward_times(synth.random_small(seed, N, D, S, tight=tight, tmax=tmax), 7 + seed, tmax)
    if comm:
        pr = synth.with_cut_bytes(pr, seed, 1000, lo=0, hi=tmax, zero_frac=0.1)
    return pr


@pytest.mark.parametrize("width,algo", [(WIDTHS[0], B.ALGO_AUTO), (WIDTHS[0], B.ALGO_SCAN), (WIDTHS[1], B.ALGO_AUTO),
                                        (1 << 41, B.ALGO_AUTO), (1 << 41, B.ALGO_SCAN)])
def test_shape_sweep_split(width, algo):
    """32-bit tables and 64-bit tables with a time bound up to 2^42 - 2 take the packed-key level
    kernel, RANNC_DP_ALGO_SCAN and larger bounds the literal one."""
    for n, (N, D, S) in enumerate(SHAPES):
        for k, tight in enumerate((1.3, 2.0, 40.0)):
            pr = _case(2900 + n, N, D, S, tight, [6, 5000][(n + k) % 2], comm=(n + k) % 3 == 0)
            if width > B.NARROW_MAX_TOTAL_TIME:
                up = 1 << (24 if width > (1 << 42) else 20)   # totals beyond 32 bits, within the bound
                for key in ("time_ns", "time_bwd_ns"):
                    pr[key] = pr[key] * up
                if "cut_bytes" in pr:
                    pr["cut_bytes"] = pr["cut_bytes"] * up
            res, sess = gpu_run([pr], max_total_time_ns=width, algo=algo)
            with sess:
                assert_results_match([pr], res)
                assert_tables_match(pr, sess, 0, args=(N <= 100))


def test_split_batch_across_device_classes():
    probs = []
    for seed in range(48):
        g = np.random.default_rng(93_000 + seed)
        N, D = int(g.integers(1, 150)), int(g.integers(1, 65))
        probs.append(_case(seed, N, D, int(g.integers(1, 14)), float(g.choice([1.2, 2.0, 9.0])),
                           int(g.choice([4, 2000])), comm=False))
    res, sess = gpu_run(probs)
    with sess:
        assert_results_match(probs, res)
        for q in (0, 5, 11, 30):
            assert_tables_match(probs[q], sess, q, args=False)
        # per-level values and the plan of a forced stage count
        Q, stride = len(probs), sess.plan_stride
        d_vals = torch.empty((Q, stride), dtype=torch.int64, device="cuda:0")
        assert B.rannc_dp_level_values(sess.h, sess.stream(), stride, d_vals) == B.OK
        lev = torch.full((Q,), 3, dtype=torch.int32, device="cuda:0")
        d_se = torch.full((Q, stride), -7, dtype=torch.int32, device="cuda:0")
        d_rp = torch.full((Q, stride), -7, dtype=torch.int32, device="cuda:0")
        assert B.rannc_dp_traceback_at(sess.h, sess.stream(), lev, stride, d_se, d_rp) == B.OK
        torch.cuda.synchronize()
        vals, se, rp = d_vals.cpu().numpy(), d_se.cpu().numpy(), d_rp.cpu().numpy()
        forced = 0
        for q, pr in enumerate(probs):
            o = oracle.solve(pr, keep_tables=True)
            N, D, L = pr["time_ns"].shape[0], pr["n_devices"], o["n_levels"]
            assert vals[q, :L].tolist() == [int(o["V"][s, N, D]) for s in range(1, L + 1)]
            assert (vals[q, L:] == INF).all()
            if L >= 3 and int(o["V"][3, N, D]) != INF:
                wse, wrp = oracle.traceback(o["arg_i"], o["arg_d"], 3, 3)
                assert np.array_equal(se[q, :3], wse) and np.array_equal(rp[q, :3], wrp), q
                assert (se[q, 3:] == -1).all()
                forced += 1
            else:
                assert (se[q] == -1).all() and (rp[q] == -1).all()
        assert forced >= 10
    # the heuristic matters somewhere in this batch: a value above the exact two-halves-equal bound is
    # not checkable at this size, but plans must differ from the min-max search's for some problem
    differs = 0
    for pr in probs[:24]:
        bare = {k: v for k, v in pr.items() if k != "time_bwd_ns"}
        bare["time_ns"] = pr["time_ns"] + pr["time_bwd_ns"]
        a, b = oracle.solve(pr), oracle.solve(bare)
        differs += not (np.array_equal(a["stage_end"], b["stage_end"]) and np.array_equal(a["replicas"], b["replicas"]))
    assert differs >= 2, differs


@pytest.mark.parametrize("algo", [B.ALGO_AUTO, B.ALGO_SCAN])
@pytest.mark.parametrize("k", [2, 3])
def test_named_configs_split(k, algo):
    """BERT-like and ResNet-like chains with a backward pass of about twice the forward time."""
    pr = synth.with_backward_times(synth.named_config(k), 23)
    res, sess = gpu_run([pr], algo=algo)
    with sess:
        assert_results_match([pr], res)
        assert_tables_match(pr, sess, 0)


def test_config4_split_full_size():
    pr = synth.with_backward_times(synth.named_config(4), 5)
    res, sess = gpu_run([pr])  # forward + backward totals still fit 32-bit tables
    with sess:
        assert_results_match([pr], res, threads=0)
        assert_tables_match(pr, sess, 0, threads=0, args=False)


def test_split_status_words_and_rejections():
    good = _case(1, 12, 4, 3, 3.0, 1000, comm=True)
    neg = dict(good); neg["time_bwd_ns"] = good["time_bwd_ns"].copy(); neg["time_bwd_ns"][7] = -2
    big = dict(good); big["time_bwd_ns"] = good["time_bwd_ns"] + (1 << 29)   # forward alone would fit
    res, sess = gpu_run([good, neg, big, good])
    with sess:
        assert list(res["status"]) == [B.PROBLEM_OK, B.PROBLEM_NEGATIVE_INPUT, B.PROBLEM_TIME_TOO_LARGE,
                                       B.PROBLEM_OK]
        for q in (1, 2):
            assert res["opt"][q] == INF and res["n_stages"][q] == 0 and (res["stage_end"][q] == -1).all()
        assert_results_match([good], {k: v[[3]] for k, v in res.items()})
        # a batch without backward times on a split handle
        hb = B.HostBatch(*[sess.batch_np[k] for k in ("n_blocks", "n_devices", "max_stages", "n_microbatches",
                                                       "mem_capacity", "block_offset")], *sess.d_in,
                         sess.batch_np["bandwidth_bytes_per_us"], sess.d_cut, None)
        assert B.rannc_dp_solve(sess.h, hb, sess.stream(), sess.d_opt, sess.d_ns) == B.INVALID_ARG
        torch.cuda.synchronize()
    res, sess = gpu_run([big], max_total_time_ns=1 << 60)
    with sess:
        assert_results_match([big], res)
    # backward times on a handle without the flag; split tables of a min-max handle
    plain = synth.random_small(1, 12, 4, 3, tight=3.0)
    res, sess = gpu_run([plain])
    with sess:
        d_b = torch.zeros(12, dtype=torch.int64, device="cuda:0")
        hb = B.HostBatch(*[sess.batch_np[k] for k in ("n_blocks", "n_devices", "max_stages", "n_microbatches",
                                                       "mem_capacity", "block_offset")], *sess.d_in, None, None, d_b)
        assert B.rannc_dp_solve(sess.h, hb, sess.stream(), sess.d_opt, sess.d_ns) == B.INVALID_ARG
        assert B.rannc_dp_read_table(sess.h, B.TABLE_MAX_FWD, 0, sess.d_se, 8, sess.stream()) == B.INVALID_ARG
        assert B.rannc_dp_read_table(sess.h, B.TABLE_COST_BWD, 0, sess.d_se, 8, sess.stream()) == B.INVALID_ARG
        torch.cuda.synchronize()
    lim = B.make_limits(1, 8, 4, 4, flags=2)
    assert B.rannc_dp_workspace_bytes(lim) == 0


FS_SPLIT = []
for seed in range(20):
    g = np.random.default_rng(71_000 + seed)
    FS_SPLIT.append((seed, int(g.integers(2, 60)), int(g.choice([1, 2, 4, 8])), int(g.integers(1, 9)),
                     int(g.choice([4, 16, 64, 256])), float(g.choice([0.6, 1.0, 2.0, 20.0])), seed % 2 == 0))


@pytest.mark.parametrize("seed,N,n_nodes,d_node,BS,tight,comm", FS_SPLIT)
def test_form_stage_on_a_split_handle(seed, N, n_nodes, d_node, BS, tight, comm):
    """The outer driver (Algorithm 2) with Algorithm 1 as printed underneath, which is the paper's
    own pipeline, with and without the send time of the cuts."""
    if d_node * max(n for n in (1, 2, 4, 8) if n <= n_nodes) > B.MAX_DEVICES:
        pytest.skip("more devices than the kernels are built for")
    c = synth.form_stage_case(seed, N, n_nodes, d_node, BS, tight=tight, tmax=60)
    g = np.random.default_rng(seed)
    tb = g.integers(0, 120, N, endpoint=True)
    os_, w = (g.integers(0, 40, N, endpoint=True), 1000) if comm else (None, 0)
    want = oracle.form_stage(c["time_per_sample_ns"], c["act_bytes_per_sample"], c["param_bytes"],
                             n_nodes, d_node, BS, c["mem_capacity"], n_threads=0,
                             cut_bytes_per_sample=os_, bandwidth_bytes_per_us=w, time_bwd_per_sample_ns=tb)
    fs = B.FormStageSession(N, n_nodes, d_node, BS, split=True)
    try:
        rc, out, se, rp = fs.run(c["time_per_sample_ns"], c["act_bytes_per_sample"], c["param_bytes"],
                                 c["mem_capacity"], os_, w, tb)
        assert rc == B.OK
        # the same handle refuses inputs without backward times
        rc2, *_ = fs.run(c["time_per_sample_ns"], c["act_bytes_per_sample"], c["param_bytes"], c["mem_capacity"])
        assert rc2 == B.INVALID_ARG
    finally:
        fs.close()
    if want is None:
        assert out.feasible == 0 and (se == -1).all()
        return
    have = {"n": out.n, "devices": out.devices, "replica_factor": out.replica_factor,
            "n_stages": out.n_stages, "n_microbatches": out.n_microbatches,
            "stage_time_ns": out.stage_time_ns, "est_iter_ns": out.est_iter_ns}
    for k, v in have.items():
        assert v == want[k], (k, v, want[k])
    S = want["n_stages"]
    assert np.array_equal(se[:S], want["stage_end"]) and np.array_equal(rp[:S], want["replicas"])
    assert (se[S:] == -1).all() and (rp[S:] == -1).all()


def test_split_64bit_packed_at_size():
    """The ResNet-like chain with times in units that need 64-bit tables, through the packed-key
    kernel of a handle whose time bound is 2^41, and through the literal kernel of a wider one."""
    pr = synth.with_backward_times(synth.named_config(3), 23)
    for key in ("time_ns", "time_bwd_ns"):
        pr[key] = pr[key] * 4096
    ra, sa = gpu_run([pr], max_total_time_ns=1 << 41)
    rb, sb = gpu_run([pr], max_total_time_ns=1 << 50)
    with sa, sb:
        assert_results_match([pr], ra)
        for k in ra:
            assert np.array_equal(ra[k], rb[k]), k
        assert_tables_match(pr, sa, 0, args=False)


# A launch with enough column chunks in its widest class (one to a chain here), weighted by the devices that its levels
# still deal with, finishes every level's winners in a launch of its own: either side of each line, chains of
# different stage counts together.
@pytest.mark.parametrize("width,D,below", [(WIDTHS[0], 57, 5), (1 << 41, 64, 4), (WIDTHS[0], 32, 12), (1 << 41, 29, 5),
                                           (WIDTHS[0], 13, 54), (1 << 41, 16, 32), (WIDTHS[0], 8, 132), (1 << 41, 7, 143)])
@pytest.mark.parametrize("apart", [0, 1])
def test_winners_in_the_next_level_or_apart(width, D, below, apart):
    Q, S = below + apart, [7, 2, 5, 3, 4]
    share = sum((D - s + 1) ** 2 for s in range(2, 8)) / (8 if D <= 8 else 16 if D <= 16 else 32 if D <= 32 else 64) ** 2 / 6
    line = {57: 4, 64: 4, 32: 10, 29: 3.5, 13: 20, 16: 20, 8: 48, 7: 34}[D]
    assert (Q * share >= line) == bool(apart)
    distinct = [_case(5100 + k, 60 + k, D, S[k], (1.5, 3.0)[k % 2], 5000, comm=D % 2 == 0) for k in range(5)]
    if width > B.NARROW_MAX_TOTAL_TIME:
        for pr in distinct:
            for key in ("time_ns", "time_bwd_ns", "cut_bytes"):
                if key in pr:
                    pr[key] = pr[key] << 20
    probs = [distinct[q % 5] for q in range(Q)]
    res, sess = gpu_run(probs, max_total_time_ns=width)
    with sess:
        want = [oracle.solve(pr) for pr in distinct]
        assert_results_match(probs, res, oracle_results=[want[q % 5] for q in range(Q)])
        for q in (1, Q - 1):
            assert_tables_match(probs[q], sess, q, args=False)
