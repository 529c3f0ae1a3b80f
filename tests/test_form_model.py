"""The method of the kernel behind the outer driver (csrc/rannc_dp_form.hip), written down from its definition: the values
of Algorithm 1 for exactly S stages on D devices from the cells that can be part of such a plan alone, against the
oracle's full tables, with one objective and with forward and backward maxima apart."""
import numpy as np
import pytest

import oracle
from paper_2103_16063_amd import synth


def _value(p, S):
    """V[S][N][D] from the live cells, or None."""
    D, M, N = p["n_devices"], p["mem_capacity"], len(p["time_ns"])
    sums = lambda k: np.concatenate(([0], np.cumsum(p[k]))).astype(object)
    T, P, A = sums("time_ns"), sums("param_bytes"), sums("act_bytes")
    TB = sums("time_bwd_ns") if "time_bwd_ns" in p else None
    C = [0] * (N + 1)
    if "cut_bytes" in p:
        for j in range(1, N):
            C[j] = -(-1000 * int(p["cut_bytes"][j - 1]) // int(p["bandwidth_bytes_per_us"]))
    K = D - S + 1
    up = lambda x, r: -(-x // r)
    fits = lambda i, j, r: P[j] - P[i] + up(A[j] - A[i], r) <= M
    reach = lambda i: max(j for j in range(i, N + 1) if j == i or fits(i, j, K))
    back = lambda j: min(i for i in range(0, j + 1) if i == j or fits(i, j, K))
    a, b = [0], [N]
    for _ in range(S):
        a.append(reach(a[-1]))
        b.append(back(b[-1]))
    if a[S] < N:
        return None
    rows = lambda s: [0] if s == 0 else [N] if s == S else range(max(s, b[S - s]), min(a[s], N - (S - s)) + 1)
    cells = {(0, 0): (0, 0, 0)}     # (row, devices) -> value, forward, backward
    for s in range(1, S + 1):
        now = {}
        for j in rows(s):
            for d in range(s, s + K):
                best = None         # the first candidate in scan order with the smallest value
                for (i, e), (_, f, g) in sorted(cells.items()):
                    if i < j and 1 <= d - e <= K and fits(i, j, d - e):
                        h = up(T[j] - T[i], d - e) + up(C[j], d - e)
                        f2 = max(f, h)
                        g2 = max(g, up(TB[j] - TB[i], d - e)) if TB is not None else 0
                        if best is None or f2 + g2 < best[0]:
                            best = (f2 + g2, f2, g2)
                if best:
                    now[j, d] = best
        cells = now
    return cells[N, D][0] if (N, D) in cells else None


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("comm", [False, True])
def test_values_of_exact_stage_counts_from_live_cells(split, comm):
    found = 0
    for seed in range(40):
        g = np.random.default_rng([seed, split, comm])
        N, D = int(g.integers(1, 11)), int(g.integers(1, 10))
        p = synth.random_small(seed, N, D, D, tight=float(g.choice([0.5, 0.9, 1.3, 4.0])))
        if comm:
            p = synth.with_cut_bytes(p, seed, 1000, lo=0, hi=1 << 16)
        if split:
            p = synth.with_backward_times(p, seed, tmax=40)
        V = oracle.solve(p, keep_tables=True)["V"]
        for S in range(max(1, D - 7), min(N, D) + 1):
            want = int(V[S][N][D])
            got = _value(p, S)
            assert got == (None if want == oracle.INF else want), (seed, S)
            found += got is not None
    assert found > 30
