"""The rule of the kernels that run Algorithm 1's levels among the cells that a bound leaves (reach_levels in
csrc/rannc_dp_reach.h), written down from its definition and compared with the oracle's full tables: for every bound from the
optimum up the levels give the optimum, its stages and the canonical plan, below it nothing; with send times, with forward and
backward maxima apart (where what a cell keeps is no minimum over plans), and with both."""
import numpy as np
import pytest

import oracle


def _levels(p, U):
    """(value, stages, ends, replicas) from the cells that U leaves, or None."""
    D, M, N = p["n_devices"], p["mem_capacity"], len(p["time_ns"])
    S = min(p["max_stages"], N, D)
    sums = lambda x: [0] + [int(v) for v in np.cumsum(x)]
    F, P, A = sums(p["time_ns"]), sums(p["param_bytes"]), sums(p["act_bytes"])
    G = sums(p["time_bwd_ns"]) if "time_bwd_ns" in p else [0] * (N + 1)
    T = [f + g for f, g in zip(F, G)]
    C = [0] * (N + 1)
    if "cut_bytes" in p:
        C[1:N] = [-(-1000 * int(o) // int(p["bandwidth_bytes_per_us"])) for o in p["cut_bytes"][:N - 1]]
    up = lambda x, r: -(-x // r)
    fits = lambda i, j, r: P[j] - P[i] + up(A[j] - A[i], r) <= M
    # first row behind which e devices take the rest, every stage's share of T within U
    back = [N]
    for e in range(1, D + 1):
        back.append(min([N] + [i for f in range(e) for i in range(back[f])
                               if T[back[f]] - T[i] <= (e - f) * U and fits(i, back[f], e - f)]))
    rows = lambda d: [N] if d == D else [i for i in range(max(1, back[D - d]), N) if T[i] <= d * U]
    before = {(0, 0): (0, 0, None)}   # (row, devices) -> forward, backward, what it comes from
    made, best = [before], None
    for s in range(1, S + 1):
        now = {}
        for d in range(1, D + 1):
            for j in rows(d):
                kept = None             # the first candidate in scan order with the smallest value
                for (i, e) in sorted(before):
                    if i < j and e < d and fits(i, j, d - e):
                        r = d - e
                        f = max(before[i, e][0], up(F[j] - F[i], r) + up(C[j], r))
                        g = max(before[i, e][1], up(G[j] - G[i], r))
                        if f + g <= U and (kept is None or f + g < kept[0]):
                            kept = (f + g, f, g, (i, e))
                if kept:
                    now[j, d] = kept[1:]
        if (N, D) in now:
            v = now[N, D][0] + now[N, D][1]
            if best is None or v < best[0]:
                best, U = (v, s), min(U, v - 1)
        made.append(now)
        before = {c: x for c, x in now.items() if c != (N, D) and x[0] + x[1] <= U}
    if best is None:
        return None
    ends, reps, c = [], [], (N, D)
    for s in range(best[1], 0, -1):
        e = made[s][c][2]
        ends.insert(0, c[0])
        reps.insert(0, c[1] - e[1])
        c = e
    return best + (ends, reps)


@pytest.mark.parametrize("form", ["", "c", "s", "cs"])
@pytest.mark.parametrize("seed", range(12))
def test_levels_among_the_cells_of_a_bound(form, seed):
    g = np.random.default_rng([seed, len(form)])
    N, D, S = int(g.integers(2, 12)), int(g.integers(1, 8)), int(g.integers(1, 7))
    top = int(g.choice([3, 40, 1000]))          # many equal values / few
    p = {"name": f"{form}_{seed}", "n_devices": D, "max_stages": S, "n_microbatches": 4, "time_ns": g.integers(0, top + 1, N),
         "param_bytes": g.integers(1, 100, N), "act_bytes": g.integers(1, 100, N)}
    if "s" in form:
        p["time_bwd_ns"] = g.integers(0, 2 * top + 1, N)
    if "c" in form:
        p["cut_bytes"], p["bandwidth_bytes_per_us"] = g.integers(0, int(g.choice([2, top, 5 * top])) + 1, N), 1000
    p["mem_capacity"] = int((p["param_bytes"].sum() + p["act_bytes"].sum()) / min(S, N, D) * g.choice([0.9, 1.1, 1.5, 4.0]))
    o = oracle.solve(p, n_threads=1)
    all_times = int(p["time_ns"].sum()) * 3 + 20 * top + 100
    if o["n_stages"] == 0:
        assert _levels(p, all_times) is None
        return
    n, opt = o["n_stages"], o["opt"]
    assert _levels(p, opt - 1) is None
    for U in (opt, opt + 1, opt + max(1, opt // 10), 2 * opt + 1, all_times + opt):
        v, s, ends, reps = _levels(p, U)
        assert (v, s) == (opt, n), (U, v, s, opt, n)
        assert ends == list(o["stage_end"][:n]) and reps == list(o["replicas"][:n]), U
