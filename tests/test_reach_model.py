"""The method of the kernel that answers a min-max search without its tables (csrc/rannc_dp_reach.hip), written down
from its definition and compared with the oracle: the bound within which D devices take the chain in at most S
stages, the fewest stages, and the canonical plan found among the cells that can complete one.  (The kernel takes the bound
of any number of stages and leaves a search for which S do not suffice there to others.)"""
import numpy as np
import pytest

import oracle


def answer(t, p, a, D, S, M):
    N = len(t)
    T, P, A = (np.concatenate(([0], np.cumsum(x))).astype(object) for x in (t, p, a))

    def stage(i, j, r, x):  # blocks i+1..j on r replicas take at most x and fit
        return T[j] - T[i] <= r * x and P[j] - P[i] + -(-(A[j] - A[i]) // r) <= M

    def reaches(x, most):  # R_s(d), s = 1..most: the last block that at most s stages on d devices reach
        levels = [[0] * (D + 1)]
        for _ in range(most):
            now = list(levels[-1])
            for e in range(D):
                i = levels[-1][e]
                for d in range(e + 1, D + 1):
                    while now[d] < N and i <= now[d] and stage(i, now[d] + 1, d - e, x):
                        now[d] += 1
            levels.append(now)
        return levels

    def fewest(x, most):
        return next((s for s, level in enumerate(reaches(x, most)) if level[D] == N), 0)

    S = min(S, N, D)
    if not fewest(T[N], S):
        return None
    lo, hi = -1, T[N]
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fewest(mid, S) else (mid, hi)
    opt, n = hi, fewest(hi, S)
    # first row behind which e devices take the rest within opt, in any number of stages
    back = [N] + [N + 1] * D
    for e in range(1, D + 1):
        back[e] = min([back[e - 1]] + [i for f in range(e) if back[f] <= N for i in range(back[f]) if stage(i, back[f], e - f, opt)])
    cells = [(d, j) for d in range(1, D) for j in range(max(1, back[D - d]), N)] + [(D, N)]
    best = {(0, 0): (0, 0)}     # fewest stages, then the smallest value of a plan with so few
    for d, j in cells:
        for (e, i), (s, v) in list(best.items()):
            if e < d and i < j and stage(i, j, d - e, opt):
                new = (s + 1, max(v, -(-(T[j] - T[i]) // (d - e))))
                best[d, j] = min(best.get((d, j), new), new)
    assert best[D, N][0] == n
    ends, reps, (d, j), x = [], [], (D, N), opt
    for s in range(n, 0, -1):   # smallest row, then fewest devices, among the candidates of the cell's value
        i, e = min((i, e) for (e, i), (k, v) in best.items() if k == s - 1 and e < d and i < j and v <= x and stage(i, j, d - e, x))
        ends.insert(0, j)
        reps.insert(0, d - e)
        (d, j), x = (e, i), best[e, i][1]
    return opt, n, ends, reps


@pytest.mark.parametrize("kind", ["plain", "equal", "one long", "zeros", "one large", "transient"])
def test_the_method_gives_the_oracles_plan(kind):
    plans = 0
    for seed in range(60):
        g = np.random.default_rng([seed, len(kind), ord(kind[0])])
        N, D, S = int(g.integers(1, 13)), int(g.integers(1, 8)), int(g.integers(1, 8))
        t, p, a = (g.integers(lo, int(g.choice([3, 12, 1000])), N).astype(np.int64) for lo in (1, 0, 0))
        if kind == "equal":
            t[:], p[:], a[:] = t[0], p[0], a[0]
        if kind == "one long":
            t[g.integers(0, N)] = 3 * t.sum()
        if kind == "zeros":
            t[g.random(N) < 0.6] = 0
        if kind == "one large":
            p[g.integers(0, N)] = p.sum() + 1
        if kind == "transient":
            a *= 40
        M = int((p.sum() + a.sum()) / max(1, min(S, D, N)) * g.choice([0.5, 0.9, 1.1, 1.5, 3.0])) + int(g.integers(0, 2))
        want = oracle.solve({"name": f"{kind}{seed}", "time_ns": t, "param_bytes": p, "act_bytes": a, "n_devices": D, "max_stages": S,
                             "n_microbatches": 1, "mem_capacity": M})
        got = answer(t, p, a, D, S, M)
        if got is None:
            assert want["n_stages"] == 0, seed
            continue
        plans += 1
        n = want["n_stages"]
        assert got == (want["opt"], n, list(want["stage_end"][:n]), list(want["replicas"][:n])), seed
    assert plans > 20
