"""The work that a user of this library has it do, as cases of stated size: single searches, sweeps of
many searches, the outer driver and the compaction step, each through the public binding with its
defaults, from inputs in hand to the plan in the caller's hands.

    listed()           the named cases
    draw(rng)          one more case of the same ranges
    prepare(case, s)   a user's session (handle, workspace) and inputs, made from the seed s
    run(state)         one pass
    work(case)         bytes and operations that no implementation of the search can do without
    tolerance(case)    all results are whole numbers
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth

MiB, GiB = 1 << 20, 1 << 30
BANDWIDTH = 100_000        # bytes per microsecond between stages (communication term)
WIDE_BOUND = 1 << 40       # ns; a 64-bit handle whose searches stay below 18 minutes
BLOCK_BYTES = 4 * 64 * MiB * math.exp(0.08)   # mean persistent bytes of a lognormal block


def _search(name, N, D, S, mem_gib, **opt):
    """One search: the chain's shape, devices, stages and memory; options: chain (how the blocks look),
    wide (64-bit handle, microbatches of 64 samples), comm (send times between stages), split
    (forward and backward maxima apart)."""
    return dict({"name": name, "kind": "search", "N": N, "D": D, "S": S, "MB": 32, "mem_gib": float(mem_gib),
                 "chain": "lognormal", "wide": False, "comm": False, "split": False}, **opt)


def _driver(name, N, nodes, per_node, batch, split=False, comm=False):
    return {"name": name, "kind": "driver", "N": N, "nodes": nodes, "per_node": per_node, "batch": batch,
            "tight": 1.3, "split": split, "comm": comm}


def listed():
    return [
        # the smallest call: a hand-sized chain on one node, nothing but latency
        _search("tiny_16", 16, 4, 4, 1.5, MB=4, chain="uniform"),
        # a 24-layer transformer on two nodes, one block per sublayer: the everyday interactive search
        _search("layers_96", 96, 16, 8, 32, chain="layers"),
        # a convolutional chain, odd sizes, with the send times between stages counted
        _search("comm_251", 251, 24, 15, 3, MB=64, chain="growing", comm=True),
        # the largest single search: fine-grained blocks of an enlarged model, memory binds
        _search("enlarged_1024", 1024, 64, 32, 32, MB=128),
        # the same on devices of 288 GB, whose memory hardly ever binds: every stage is a candidate
        _search("roomy_1024", 1024, 64, 32, 288, MB=128),
        # microbatches of 64 samples: times beyond 32 bits, sizes that divide nothing
        _search("wide_701", 701, 48, 24, 48, wide=True),
        # forward and backward maxima kept apart (Algorithm 1 as printed), 32 devices
        _search("split_256", 256, 32, 16, 24, MB=64, split=True),
        # a what-if sweep: thousands of chains, device counts and microbatch counts in one call
        {"name": "sweep_2048", "kind": "batch", "Q": 2048, "N": 128, "ragged": False, "d_max": 64, "S": 16,
         "mem_gib": 16.0},
        # the whole partitioner's question, "how do I split this model on this cluster": node
        # counts, stage counts and microbatch counts tried, at the usual number of blocks ...
        _driver("driver_32", 32, 4, 8, 256),
        # ... on a finer chain ...
        _driver("driver_512", 512, 4, 8, 256),
        # ... and with forward and backward times apart
        _driver("driver_split_96", 96, 4, 8, 256, split=True),
        # the step in front: the sublayers of a very deep model merged into the blocks of a search
        {"name": "compact_15000", "kind": "compact", "G": 15000, "k": 32, "tight": 4.0},
    ]


def _between(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "batch", "batch", "driver", "driver", "compact"])
    if kind == "search":
        split = rng.random() < 0.2
        N = _between(rng, 8, 400 if split else 1024)
        D = _between(rng, 2, 32 if split else 64)
        S = _between(rng, 2, 32)
        # capacity as a multiple of an even share of the chain over the stages
        share = N * (BLOCK_BYTES + 40 * MiB) / min(S, D, N) / GiB
        wide = not split and rng.random() < 0.25
        comm = rng.random() < 0.25
        c = _search("", N, D, S, round(share * math.exp(rng.uniform(math.log(1.5), math.log(20))), 3),
                    MB=rng.choice([8, 16, 32, 64, 128]), wide=wide, comm=comm, split=split)
    elif kind == "batch":
        N = _between(rng, 16, 160)
        Q = _between(rng, 8, min(2048, 2048 * 128 * 128 // (N * N)))
        S = _between(rng, 4, 16)
        d_max = rng.choice([8, 16, 32, 64])
        share = N * (BLOCK_BYTES + 40 * MiB) / min(S, 8) / GiB
        c = {"name": "", "kind": "batch", "Q": Q, "N": N, "ragged": rng.random() < 0.7, "d_max": d_max, "S": S,
             "mem_gib": round(share * rng.uniform(1.5, 8.0), 3)}
    elif kind == "driver":
        split = rng.random() < 0.3
        N = _between(rng, 12, 128 if split else 512)
        c = _driver("", N, rng.choice([1, 2, 3, 4]), rng.choice([4, 6, 8]), _between(rng, 16, 512), split,
                    rng.random() < 0.3)
        # capacity as a multiple of an even share over all devices; a stage holds at least one whole block
        per_block = c["nodes"] * c["per_node"] / N
        c["tight"] = round(math.exp(rng.uniform(math.log(2), math.log(8))) * max(1.0, 1.5 * per_block), 3)
    else:
        c = {"name": "", "kind": "compact", "G": _between(rng, 64, 15000), "k": _between(rng, 8, 128),
             "tight": round(math.exp(rng.uniform(math.log(2), math.log(16))), 3)}
    del c["name"]
    return c


def _chain(case, seed):
    """The blocks of one search."""
    N, D, S, MB, M = case["N"], case["D"], case["S"], case["MB"], int(case["mem_gib"] * GiB)
    if case["chain"] == "uniform":
        p = synth.tiny_chain(seed, N=N, D=D, S=S, MB=MB, M=M)
    elif case["chain"] == "layers":
        p = synth.bert_like_chain(seed, layers=N // 4, D=D, S=S, MB=MB, M=M)
    elif case["chain"] == "growing":
        p = synth.resnet_like_chain(N=N, D=D, S=S, MB=MB, M=M)
        jitter = np.random.default_rng(seed).uniform(0.9, 1.1, (3, N))
        for row, key in zip(jitter, ("time_ns", "param_bytes", "act_bytes")):
            p[key] = (p[key] * row).astype(np.int64)
    else:
        p = synth.enlarged_transformer_chain(seed, N=N, D=D, S=S, MB=MB, M=M)
    if case["wide"]:
        p["time_ns"] = p["time_ns"] * 64
    if case["comm"]:
        p = synth.with_cut_bytes(p, seed + 1, BANDWIDTH, lo=1 * MiB, hi=64 * MiB)
    if case["split"]:
        p = synth.with_backward_times(p, seed + 2)
    return p


def _sweep(case, seed):
    """The searches of a sweep: chains of their own, device counts up to d_max, the sizes of a ragged one
    within a factor of two."""
    g = np.random.default_rng(seed)
    out = []
    for q in range(case["Q"]):
        N = int(g.integers(max(2, (2 * case["N"]) // 3), (4 * case["N"]) // 3, endpoint=True)) if case["ragged"] else case["N"]
        D = int(g.choice([d for d in (8, 16, 32, 64) if d <= case["d_max"]]))
        if case["ragged"]:
            D -= int(g.integers(0, 4))
        out.append(synth.enlarged_transformer_chain(int(g.integers(1 << 40)), N=N, D=D, S=case["S"],
                                                    MB=int(g.choice([8, 16, 32, 64])), M=int(case["mem_gib"] * GiB)))
    return out


class _Opened(dict):
    """A prepared case; gives its session back when the program is done with it."""

    def __del__(self):
        if "session" in self:
            self["session"].close()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "search":
        bound = WIDE_BOUND if case["wide"] else B.NARROW_MAX_TOTAL_TIME
        session = B.Session(synth.concat_batch([_chain(case, seed)]), max_total_time_ns=bound)
        return _Opened(kind=kind, session=session)
    if kind == "batch":
        return _Opened(kind=kind, session=B.Session(synth.concat_batch(_sweep(case, seed))))
    if kind == "driver":
        c = synth.form_stage_case(seed, case["N"], case["nodes"], case["per_node"], case["batch"], tight=case["tight"],
                                  tmax=2000, layered=True)
        more = {}
        if case["comm"]:
            g = np.random.default_rng(seed + 1)
            more["cut_bytes_per_sample"] = g.integers(1 << 12, 1 << 18, case["N"], endpoint=True)
            more["bandwidth_bytes_per_us"] = BANDWIDTH
        if case["split"]:
            more["time_bwd_per_sample_ns"] = synth.with_backward_times(
                {"time_ns": c["time_per_sample_ns"], "name": c["name"]}, seed + 2)["time_bwd_ns"]
        fs = B.FormStageSession(case["N"], case["nodes"], case["per_node"], case["batch"], split=case["split"])
        return _Opened(kind=kind, session=fs, more=more, inputs=(
            c["time_per_sample_ns"], c["act_bytes_per_sample"], c["param_bytes"], c["mem_capacity"]))
    # sublayers of a deep model: lognormal times and sizes, capacity as a multiple of an even share
    G = case["G"]
    g = np.random.default_rng(seed)
    t = np.floor(g.lognormal(math.log(2e4), 0.8, G)).astype(np.int64)
    p = np.floor(g.lognormal(math.log(8 * MiB), 0.8, G)).astype(np.int64)
    a = g.integers(1 * MiB, 8 * MiB, G, endpoint=True)
    M = int(case["tight"] * (int(p.sum()) + int(a.sum())) / case["k"])
    dev = torch.device("cuda:0")
    ins = [torch.from_numpy(x).to(dev) for x in (t, p, a)]
    nbytes = B.rannc_dp_compact_workspace_bytes(G)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    n = torch.zeros(1, dtype=torch.int32, device=dev)
    end = torch.full((G,), -1, dtype=torch.int32, device=dev)   # entries behind the last block are not written
    outs = [torch.zeros(G, dtype=torch.int64, device=dev) for _ in range(3)]
    status = torch.zeros(1, dtype=torch.int32, device=dev)
    return _Opened(kind=kind, G=G, k=case["k"], M=M, ins=ins, ws=ws, nbytes=nbytes, n=n, end=end, outs=outs, status=status)


def run(state):
    kind = state["kind"]
    if kind in ("search", "batch"):
        return state["session"].run()   # optimum, stage count, plan: on the host, as the README's example
    if kind == "driver":
        rc, out, stage_end, replicas = state["session"].run(*state["inputs"], **state["more"])
        return {"rc": rc, "feasible": out.feasible, "n": out.n, "devices": out.devices,
                "replica_factor": out.replica_factor, "n_stages": out.n_stages, "n_microbatches": out.n_microbatches,
                "stage_time_ns": out.stage_time_ns, "est_iter_ns": out.est_iter_ns, "stage_end": stage_end,
                "replicas": replicas}
    s = state
    rc = B.rannc_dp_compact(torch.cuda.current_stream().cuda_stream, s["G"], s["k"], 0, s["M"], *s["ins"], s["ws"],
                            s["nbytes"], s["n"], s["end"], *s["outs"], s["status"])
    return {"rc": rc, "n_blocks": s["n"], "block_end": s["end"], "time": s["outs"][0], "param": s["outs"][1],
            "act": s["outs"][2], "status": s["status"]}


def _ops(N, D, S, span, split):
    """Operations of one search whose stages span at most `span` blocks: per candidate stage and level the
    D log2 D + D comparisons of a sorted merge and the D stage times; with the two objectives apart every pair
    of replica counts, seven operations each."""
    w = min(float(N), max(1.0, span))
    stages = w * N - w * w / 2
    levels = max(1, min(S, N, D) - 1)
    return stages * levels * (7.0 * D * D / 2 if split else D * (math.log2(max(2, D)) + 3.0))


def work(case):
    kind = case["kind"]
    if kind == "search":
        N, D, S = case["N"], case["D"], case["S"]
        arrays = 3 + case["comm"] + case["split"]
        return {"bytes": 8 * N * arrays + 24 + 8 * min(S, N, D),
                "flops": _ops(N, D, S, case["mem_gib"] * GiB / BLOCK_BYTES, case["split"])}
    if kind == "batch":
        ds = [d for d in (8, 16, 32, 64) if d <= case["d_max"]]
        span = case["mem_gib"] * GiB / BLOCK_BYTES
        return {"bytes": case["Q"] * (24 * case["N"] + 24 + 8 * case["S"]),
                "flops": case["Q"] / len(ds) * sum(_ops(case["N"], d, case["S"], span, False) for d in ds)}
    if kind == "driver":
        N, flops, n = case["N"], 0.0, 1
        while n <= case["nodes"]:
            mb, D = 1, case["per_node"] * n
            while mb <= case["batch"] // (case["nodes"] // n):
                flops += _ops(N, D, D, N, case["split"])
                mb *= 2
            n *= 2
        return {"bytes": 8 * N * (3 + case["comm"] + case["split"]) + 48 + 8 * case["per_node"] * case["nodes"], "flops": flops}
    return {"bytes": 24 * case["G"] + 28 * case["k"] + 8, "flops": case["G"] * math.log2(max(2, case["G"]))}


def tolerance(case):
    return "exact"   # whole nanoseconds, bytes, counts and positions
