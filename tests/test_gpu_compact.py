"""GPU parity of the compaction step of the block-level phase (Sec. III-B) against the CPU oracle,
and the hand-over of its result, still on the device, to the stage-level search."""
import numpy as np
import pytest
import torch

import oracle
from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def gpu_compact(t, p, a, k, M, walks=0):
    G = len(t)
    d_in = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.int64)).to(DEV) for x in (t, p, a)]
    nbytes = B.rannc_dp_compact_workspace_bytes(G)
    assert nbytes > 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    d_n = torch.full((1,), -5, dtype=torch.int32, device=DEV)
    d_st = torch.full((1,), -5, dtype=torch.int32, device=DEV)
    d_end = torch.full((G,), -5, dtype=torch.int32, device=DEV)
    d_out = [torch.full((G,), -5, dtype=torch.int64, device=DEV) for _ in range(3)]
    rc = B.rannc_dp_compact(torch.cuda.current_stream().cuda_stream, G, k, walks, M, *d_in, ws, nbytes, d_n,
                            d_end, *d_out, d_st)
    torch.cuda.synchronize()
    return rc, int(d_n.item()), int(d_st.item()), d_end, d_out


CASES = []
for seed in range(60):
    g = np.random.default_rng(seed)
    G = int(g.integers(1, 200))
    CASES.append((seed, G, int(g.integers(1, G + 3)), int(g.choice([0, 60, 150, 400, 10**9]))))
CASES += [(100, 1500, 96, 3000), (101, 1600, 32, 10**9), (102, 1601, 700, 2500), (103, 5000, 128, 4000),
          (104, 3000, 1, 10**9), (105, 2048, 5, 10**9), (106, 2049, 5, 600), (107, 4100, 9, 10**9),
          (108, 9000, 40, 20000)]  # around and beyond the sizes whose state fits LDS and whose listing is a rank sort


@pytest.mark.parametrize("seed,G,k,M", CASES)
def test_compact_matches_the_oracle(seed, G, k, M):
    g = np.random.default_rng(10_000 + seed)
    t = g.integers(0, 20, G) if seed % 2 else g.integers(0, 10**6, G)   # many equal times / few
    p, a = g.integers(0, 50, G), g.integers(0, 50, G)
    for walks in (0, 1, 3):   # until k groups or a walk without merges; one walk; at most three
        rc, n, st, d_end, d_out = gpu_compact(t, p, a, k, M, walks)
        assert rc == B.OK and st == B.PROBLEM_OK
        end, tt, pp, aa = oracle.compact(t, p, a, k, M, max_passes=walks)
        assert n == len(end), (walks, n, len(end))
        assert np.array_equal(d_end.cpu().numpy()[:n], end)
        for have, want in zip(d_out, (tt, pp, aa)):
            assert np.array_equal(have.cpu().numpy()[:n], want)
        assert (d_end.cpu().numpy()[n:] == -5).all()     # nothing written behind the result
        if walks == 0 and M == 10**9:
            assert n == min(k, G)                        # memory never refuses: k blocks are reached


# the three layouts of the kernel's state (all in LDS, times in LDS, all in the workspace) at their
# edges, on chains whose turns are independent (random), strictly one after the other (ascending,
# descending) or decided by position alone (equal), with a walk that stops at k in its middle
@pytest.mark.parametrize("G", [1, 2, 63, 64, 65, 257, 1600, 1601, 16384, 16385, 65535])
@pytest.mark.parametrize("order", ["random", "ascending", "descending", "equal"])
def test_compact_state_layouts(G, order):
    if G > 20000 and order in ("ascending", "descending"):
        G = 17000   # one turn per round: keep it short
    g = np.random.default_rng(G)
    t = {"random": g.integers(0, 1 << 40, G), "ascending": np.arange(G) * 3, "descending": np.arange(G)[::-1] * 3,
         "equal": np.full(G, 7)}[order]
    p, a = g.integers(0, 50, G), g.integers(0, 50, G)
    for k, M, walks in ((1, 10**9, 0), (max(1, (3 * G) // 4), 10**9, 0), (max(1, G // 3), 130, 2)):
        rc, n, st, d_end, d_out = gpu_compact(t, p, a, k, M, walks)
        assert rc == B.OK and st == B.PROBLEM_OK
        end, tt, pp, aa = oracle.compact(t, p, a, k, M, max_passes=walks)
        assert n == len(end) and np.array_equal(d_end.cpu().numpy()[:n], end)
        for have, want in zip(d_out, (tt, pp, aa)):
            assert np.array_equal(have.cpu().numpy()[:n], want)


# walks in windows of 63 groups, and the walks of long chains that have a launch of their own: chains on which every
# window is large enough (random), too small in a few places (runs of ascending and descending times among random
# ones), and everywhere (a zigzag that rises slowly: each turn waits for the one two places before it)
@pytest.mark.parametrize("G", [17, 62, 63, 64, 80, 96, 700, 1600, 1601, 2048, 5003, 16384, 16385, 30001])
@pytest.mark.parametrize("order", ["random", "runs", "zigzag"])
def test_compact_windows(G, order):
    if G > 16384 and order == "zigzag":
        G = 16900
    g = np.random.default_rng(7 * G)
    t = g.integers(0, 1 << 30, G)
    if order == "runs":
        for at in g.integers(0, G, max(1, G // 2000)):
            n = min(int(g.integers(30, 200)), G - at)
            t[at:at + n] = (np.arange(n) if g.integers(2) else n - np.arange(n)) * 1000
    elif order == "zigzag":
        t = np.arange(G) * 5 + np.where(np.arange(G) % 2, 7, 0)
    p, a = g.integers(0, 50, G), g.integers(0, 50, G)
    for k, M, walks in ((max(1, G // 40), 10**9, 0), (5, 10**9, 1), (5, 10**9, 2), (max(1, (2 * G) // 5), 10**9, 0), (8, 150, 0),
                        (3, 0, 0)):
        rc, n, st, d_end, d_out = gpu_compact(t, p, a, k, M, walks)
        assert rc == B.OK and st == B.PROBLEM_OK
        end, tt, pp, aa = oracle.compact(t, p, a, k, M, max_passes=walks)
        assert n == len(end) and np.array_equal(d_end.cpu().numpy()[:n], end), (k, M, walks)
        for have, want in zip(d_out, (tt, pp, aa)):
            assert np.array_equal(have.cpu().numpy()[:n], want)


@pytest.mark.parametrize("G,k,walks", [(1700, 1650, 0), (5000, 1601, 0), (15000, 1000, 0), (15000, 2500, 0), (16384, 40, 1), (16385, 40, 1), (30001, 1500, 0),
                                       (30001, 7, 2), (65535, 9000, 0), (65535, 5, 3), (65535, 5, 1)])
@pytest.mark.parametrize("order", ["random", "runs"])
def test_compact_long_chains_to_many_blocks(G, k, walks, order):
    """The last walk with a launch of its own leaves more groups than one workgroup holds in LDS: what k or the limit on the walks leaves."""
    g = np.random.default_rng(G + k)
    t, p, a = g.integers(0, 1 << 30, G), g.integers(0, 50, G), g.integers(0, 50, G)
    if order == "runs":
        for at in g.integers(0, G - 100, 3):
            t[at:at + 100] = np.arange(100) * 1000
    for M in (10**9, 400):
        rc, n, st, d_end, d_out = gpu_compact(t, p, a, k, M, walks)
        assert rc == B.OK and st == B.PROBLEM_OK
        end, tt, pp, aa = oracle.compact(t, p, a, k, M, max_passes=walks)
        assert n == len(end) and np.array_equal(d_end.cpu().numpy()[:n], end), M
        for have, want in zip(d_out, (tt, pp, aa)):
            assert np.array_equal(have.cpu().numpy()[:n], want)


@pytest.mark.parametrize("G", [1700, 9000])
def test_compact_refuses_long_chains_that_overflow(G):
    """The sums of a long chain are made by many workgroups: each kind of input, at either end of the chain."""
    for at in (0, G // 2, G - 1):
        for which, value, want in ((0, -1, B.PROBLEM_NEGATIVE_INPUT), (1, -5, B.PROBLEM_NEGATIVE_INPUT), (2, -1, B.PROBLEM_NEGATIVE_INPUT),
                                   (0, 1 << 62, B.PROBLEM_SUM_OVERFLOW), (1, (1 << 62) - 1000, B.PROBLEM_SUM_OVERFLOW),
                                   (2, (1 << 62) - 1, B.PROBLEM_SUM_OVERFLOW)):
            arrays = [np.full(G, 3) for _ in range(3)]
            arrays[which][at] = value
            rc, n, st, *_ = gpu_compact(*arrays, 20, 10**9)
            assert rc == B.OK and st == want and n == 0, (at, which, value)
    arrays = [np.full(G, 3) for _ in range(3)]
    arrays[1][0], arrays[2][G - 1] = 1 << 61, 1 << 61   # neither alone
    assert gpu_compact(*arrays, 20, 10**9)[2] == B.PROBLEM_SUM_OVERFLOW
    arrays[2][G - 1] = (1 << 61) - 6 * G
    rc, n, st, *_ = gpu_compact(*arrays, 20, (1 << 62) - 1)
    assert rc == B.OK and st == B.PROBLEM_OK and n == 20


def test_compact_status_and_rejections():
    t, p, a = np.array([3, 1, 2]), np.array([1, 1, 1]), np.array([1, 1, 1])
    neg = t.copy(); neg[1] = -1
    rc, n, st, *_ = gpu_compact(neg, p, a, 2, 100)
    assert rc == B.OK and st == B.PROBLEM_NEGATIVE_INPUT and n == 0
    big = np.array([1 << 61, 1 << 61, 5])
    rc, n, st, *_ = gpu_compact(t, big, a, 2, 100)
    assert rc == B.OK and st == B.PROBLEM_SUM_OVERFLOW and n == 0
    assert B.rannc_dp_compact_workspace_bytes(0) == 0 and B.rannc_dp_compact_workspace_bytes(70000) == 0
    d = torch.zeros(3, dtype=torch.int64, device=DEV)
    di = torch.zeros(3, dtype=torch.int32, device=DEV)
    ws = torch.empty(4096, dtype=torch.uint8, device=DEV)
    s = torch.cuda.current_stream().cuda_stream
    assert B.rannc_dp_compact(s, 3, 0, 0, 5, d, d, d, ws, 4096, di, di, d, d, d, di) == B.INVALID_ARG
    assert B.rannc_dp_compact(s, 3, 2, 0, -1, d, d, d, ws, 4096, di, di, d, d, d, di) == B.INVALID_ARG
    assert B.rannc_dp_compact(s, 3, 2, -1, 5, d, d, d, ws, 4096, di, di, d, d, d, di) == B.INVALID_ARG
    assert B.rannc_dp_compact(s, 3, 2, 0, 5, d, d, d, ws, 8, di, di, d, d, d, di) == B.WORKSPACE_TOO_SMALL
    assert B.rannc_dp_compact(s, 3, 2, 0, 5, d, None, d, ws, 4096, di, di, d, d, d, di) == B.INVALID_ARG
    torch.cuda.synchronize()


def test_compaction_feeds_the_search_on_the_device():
    """400 fine-grained groups -> compaction to 96 blocks (a single walk would end at 158; repeated
    walks reach 96) -> stage-level search, the block arrays never leaving the device; the same two
    steps on the oracle give the same plan."""
    fine = synth.enlarged_transformer_chain(seed=21, N=400, D=16, S=8, MB=32, M=48 << 30)
    t, p, a = fine["time_ns"], fine["param_bytes"], fine["act_bytes"]
    k, M = 96, fine["mem_capacity"]
    rc, n, st, d_end, d_out = gpu_compact(t, p, a, k, M)
    assert rc == B.OK and st == B.PROBLEM_OK
    end, tt, pp, aa = oracle.compact(t, p, a, k, M)
    assert n == len(end) == k and np.array_equal(d_end.cpu().numpy()[:n], end)
    assert len(oracle.compact(t, p, a, k, M, max_passes=1)[0]) == 158
    # search over the n blocks, inputs = the compaction's device arrays
    lim = B.make_limits(1, n, 16, 8)
    hb = B.HostBatch([n], [16], [8], [32], [M], [0, n], *[x[:n] for x in d_out])
    nbytes = B.rannc_dp_workspace_bytes_for(lim, hb)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    rc, h = B.rannc_dp_create(lim, ws, nbytes)
    assert rc == B.OK
    try:
        d_opt = torch.empty(1, dtype=torch.int64, device=DEV)
        d_ns = torch.empty(1, dtype=torch.int32, device=DEV)
        d_se = torch.empty((1, 8), dtype=torch.int32, device=DEV)
        d_rp = torch.empty((1, 8), dtype=torch.int32, device=DEV)
        s = torch.cuda.current_stream().cuda_stream
        assert B.rannc_dp_solve(h, hb, s, d_opt, d_ns) == B.OK
        assert B.rannc_dp_traceback(h, s, 8, d_se, d_rp) == B.OK
        torch.cuda.synchronize()
    finally:
        B.rannc_dp_destroy(h)
    blocks = {"name": "compacted", "time_ns": tt, "param_bytes": pp, "act_bytes": aa, "n_devices": 16,
              "max_stages": 8, "n_microbatches": 32, "mem_capacity": M}
    o = oracle.solve(blocks, n_threads=0)
    assert int(d_opt.item()) == o["opt"] and int(d_ns.item()) == o["n_stages"] and o["n_stages"] >= 1
    assert np.array_equal(d_se.cpu().numpy()[0], o["stage_end"]) and np.array_equal(d_rp.cpu().numpy()[0], o["replicas"])


def test_long_chain_recorded_and_replayed():
    """The launches of a long chain in a captured graph, replayed on other inputs (whose windows may be too small) with eager work
    in between."""
    G, k = 5003, 40
    d_in = [torch.zeros(G, dtype=torch.int64, device=DEV) for _ in range(3)]
    nbytes = B.rannc_dp_compact_workspace_bytes(G)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    d_n, d_st = (torch.full((1,), -5, dtype=torch.int32, device=DEV) for _ in range(2))
    d_end = torch.full((G,), -5, dtype=torch.int32, device=DEV)
    d_out = [torch.full((G,), -5, dtype=torch.int64, device=DEV) for _ in range(3)]
    M = 10**9
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        assert B.rannc_dp_compact(torch.cuda.current_stream().cuda_stream, G, k, 0, M, *d_in, ws, nbytes, d_n, d_end, *d_out, d_st) == B.OK
    for seed in range(4):
        g = np.random.default_rng(seed)
        t, p, a = g.integers(0, 1 << 30, G), g.integers(0, 50, G), g.integers(0, 50, G)
        if seed == 2:
            t[1000:1200] = np.arange(200) * 1000
        for x, y in zip(d_in, (t, p, a)):
            x.copy_(torch.from_numpy(y))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        end, tt, pp, aa = oracle.compact(t, p, a, k, M)
        n = int(d_n.item())
        assert int(d_st.item()) == B.PROBLEM_OK and n == len(end) and np.array_equal(d_end.cpu().numpy()[:n], end)
        for have, want in zip(d_out, (tt, pp, aa)):
            assert np.array_equal(have.cpu().numpy()[:n], want)
