"""rannc_dp_solve_to_host (solve, plan recovery and the results in host memory as one call) against the
two calls it stands for, around the batch size up to which a batch runs as one group and writes its
results to host memory itself."""
import numpy as np
import pytest
import torch

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match

pytestmark = pytest.mark.gpu


def _mixed(Q):
    g = np.random.default_rng(Q)
    out = []
    for q in range(Q):
        N = int(g.integers(1, 140))
        p = synth.random_small(600 + q, N, int(g.choice([1, 5, 8, 13, 16, 31, 32, 48, 64])), int(g.integers(1, 9)),
                               tight=float(g.choice([0.6, 1.2, 3.0, 50.0])))
        if q % 11 == 5:
            p["act_bytes"] = p["act_bytes"].copy()
            p["act_bytes"][N // 2] = -1    # a flagged search among good ones
        out.append(p)
    return out


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("Q", [1, 2, 63, 64, 65])
def test_same_as_solve_and_traceback(Q, split):
    probs = _mixed(Q)
    if split:
        probs = [synth.with_backward_times(p, 3, tmax=50) for p in probs]
    with B.Session(synth.concat_batch(probs)) as s:
        for _ in range(3):   # the second and third call reuse staging memory and mirror
            res = s.run()
        s.d_opt.fill_(-3); s.d_se.fill_(-3)
        s.solve()
        s.traceback()
        torch.cuda.synchronize()
        for key, t in (("opt", s.d_opt), ("est_iter_ns", s.d_est), ("n_stages", s.d_ns), ("status", s.d_status),
                       ("stage_end", s.d_se), ("replicas", s.d_rp)):
            assert np.array_equal(res[key], t.cpu().numpy()), key
        good = [q for q in range(Q) if res["status"][q] == B.PROBLEM_OK]
        assert len(good) < Q or Q < 6
        if not split:
            assert_results_match([probs[q] for q in good], {k: v[good] for k, v in res.items()})


def test_rejections():
    with B.Session(synth.concat_batch([synth.random_small(1, 20, 4, 3)])) as s:
        n = s._out_host.numel()
        call = lambda **k: B.rannc_dp_solve_to_host(s.h, s.hb, s.stream(), k.get("stride", s.plan_stride),
                                                    k.get("d", s._out_dev), k.get("h", s._out_host), k.get("n", n))
        assert call() == B.OK
        assert call(n=n - 1) == B.INVALID_ARG
        assert call(stride=s.plan_stride - 1) == B.INVALID_ARG
        assert call(d=None) == B.INVALID_ARG and call(h=None) == B.INVALID_ARG
        assert call(d=s._out_dev.data_ptr() + 4) == B.INVALID_ARG
        assert B.rannc_dp_solve_to_host(None, s.hb, s.stream(), 4, s._out_dev, s._out_host, n) == B.INVALID_ARG


def test_few_searches_in_a_workspace_sized_for_many():
    """A workspace sized for 65 searches at their own device-count classes holds 61 of them although one
    group of them, padded to the widest class, would not fit: the classes then run apart."""
    narrow = [synth.random_small(700 + q, 100, 8, 8, tight=3.0) for q in range(64)]
    probs = narrow + [synth.random_small(790, 20, 64, 8, tight=3.0)]
    few = probs[4:]
    with B.Session(synth.concat_batch(probs)) as big, B.Session(synth.concat_batch(few)) as own:
        assert own.ws_bytes > big.ws_bytes      # the padded layout
        want = own.run()
        n = own._out_host.numel()
        rc = B.rannc_dp_solve_to_host(big.h, own.hb, big.stream(), own.plan_stride, own._out_dev, own._out_host, n)
        assert rc == B.OK
        got = dict(zip(("opt", "est_iter_ns", "n_stages", "status", "stage_end", "replicas"), own._h_views))
        for key, v in got.items():
            assert np.array_equal(v, want[key]), key
        assert_results_match(few, want)


def test_results_of_another_layout_are_no_completion():
    """The word that says a call of one search is done lies where a call of seven searches left its last
    optimum; an optimum equal to the call's number must not end the wait."""
    seven = [synth.random_small(800 + q, 1, 1, 1) for q in range(7)]
    one = [synth.random_small(810, 1, 1, 1)]
    for p in seven + one:
        p["mem_capacity"] = 1 << 50
    seven[6]["time_ns"] = np.array([2], np.int64)    # its optimum: the number of the second call
    one[0]["time_ns"] = np.array([77], np.int64)
    with B.Session(synth.concat_batch(seven)) as s, B.Session(synth.concat_batch(one)) as o:
        assert s.run()["opt"][6] == 2
        rc = B.rannc_dp_solve_to_host(s.h, o.hb, s.stream(), 1, o._out_dev, o._out_host, o._out_host.numel())
        assert rc == B.OK
        assert_results_match(one, dict(zip(("opt", "est_iter_ns", "n_stages", "status", "stage_end", "replicas"),
                                           o._h_views)))


def _device_mappings():
    with open("/proc/self/maps") as f:
        return sum("/dev/dri/" in line for line in f)


@pytest.mark.parametrize("Q", [1, 64])
def test_first_call_of_a_handle_allocates_no_pinned_memory(Q):
    """What hipHostMalloc hands out is a mapping of the device file; a first call that makes one waits for it."""
    probs = [synth.random_small(820 + q, 40, 16, 6, tight=2.0) for q in range(Q)]
    with B.Session(synth.concat_batch(probs)) as s:
        s.run()                    # (whatever the process does once is behind us)
    with B.Session(synth.concat_batch(probs)) as s:
        before = _device_mappings()
        res = s.run()
        assert before > 0 and _device_mappings() == before
        assert_results_match(probs, res)


def test_plan_strides_beyond_the_longest_plan():
    probs = [synth.random_small(830 + q, 40, 16, 6, tight=2.0) for q in range(3)]
    with B.Session(synth.concat_batch(probs)) as s:
        want = s.run()
        for stride in (6, 70, 300, 100, 6):      # the mirror grows twice, and serves smaller strides after
            n = 3 * 16 + 16 + 16 + 2 * 3 * 4 * stride
            d = torch.empty(n // 8, dtype=torch.int64, device="cuda:0")
            h = torch.zeros(n // 8, dtype=torch.int64)
            assert B.rannc_dp_solve_to_host(s.h, s.hb, s.stream(), stride, d, h, n) == B.OK
            w = h.numpy()
            assert np.array_equal(w[:3], want["opt"]) and np.array_equal(w[3:6], want["est_iter_ns"])
            plans = w[10:].view(np.int32).reshape(2, 3, stride)
            for key, plan in zip(("stage_end", "replicas"), plans):
                assert np.array_equal(plan[:, :6], want[key]) and (plan[:, 6:] == -1).all(), (stride, key)
