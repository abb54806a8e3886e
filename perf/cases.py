"""Timed cases of the evaluation, early-stop and search entry points.

Each case is one call (or the short sequence of calls) a planner makes on resident candidates.
Profile tables are drawn in the style of ``paper_2609_06086_amd/workloads.py`` (tens of layers,
device types up to about 3x apart in speed, memory caps of a few stages' footprint), from the
seed.  Every output is a whole number, so every tolerance is exact.
"""
import math

import numpy as np
import torch

from paper_2609_06086_amd import poseidon as P
from paper_2609_06086_amd.workloads import Problem

WARM = 500        # warm-up samples that set the first bound of the early stop and the search (paper, Sec. 4.2.3)
SCHED = {"1f1b": 0, "eager": 1, "interleaved": 2}


def _case(name, call, L, S, M, T, count, sched="1f1b", V=1, types="digits", rows=0, mode="list", allreduce=False,
          slower=30, **more):
    """call: eval | noalloc | bounded | search.  types: how stages get device types: one fixed row ("fixed"), a
    table of `rows` rows ("table") or every base-T digit row ("digits").  slower: the slowest type's layer time
    over the fastest's, in tenths."""
    c = dict(call=call, L=L, S=S, M=M, T=T, count=count, sched=sched, V=V, types=types, rows=rows, mode=mode,
             allreduce=allreduce, slower=slower, cap_lo=3.2, cap_hi=13.0, ridge=False, chunk=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a planner's smallest question: a toy model, every configuration; the call's latency is all there is
        _case("exhaustive_l8_s2", "eval", 8, 2, 4, 2, 28, mode="range", slower=20, cap_lo=2.7, cap_hi=2.8),
        # a small model on 4 stages, every configuration, still bound by launches
        _case("exhaustive_l32_s4", "eval", 32, 4, 16, 2, 71920, mode="range", slower=16, cap_hi=6.6),
        # every composition of a mid-size model for one placement of the device types
        _case("exhaustive_l48_s8", "eval", 48, 8, 32, 2, 62891499, mode="range", types="fixed", slower=20, cap_lo=3.5,
              cap_hi=10.6),
        # a large sampled sweep over compositions and device placements
        _case("sampled_l80_s8", "eval", 80, 8, 64, 3, 1 << 26, slower=26, cap_lo=4.2, cap_hi=12.8),
        # the deepest pipeline, sampled: the headline benchmark's shape
        _case("sampled_l126_s16", "eval", 126, 16, 128, 4, 1 << 24, types="fixed", cap_lo=4.0, cap_hi=16.2),
        # the 8-stage sweep with data-parallel gradient all-reduce nodes
        _case("sampled_l80_s8_allreduce", "eval", 80, 8, 64, 3, 1 << 24, allreduce=True, slower=26, cap_lo=4.2,
              cap_hi=12.8),
        # the same deep pipeline under the Eager 1F1B schedule
        _case("eager_l126_s16", "eval", 126, 16, 128, 4, 1 << 24, sched="eager", types="fixed", cap_lo=4.0, cap_hi=16.2),
        # and under Interleaved 1F1B, 2 model chunks on each of 8 devices
        _case("interleaved_l126_s16", "eval", 126, 16, 128, 4, 1 << 24, sched="interleaved", V=2, types="fixed",
              cap_lo=2.0, cap_hi=8.1),
        # a serving loop that may not allocate: odd sizes, a table of allowed placements, a ragged end
        _case("noalloc_l61_s11_ragged", "noalloc", 61, 11, 37, 5, 1000003, types="table", rows=23, mode="range",
              slower=25),
        # the search's screening pass: warm-up samples set a bound, Eq. 2 discards most of the list
        _case("early_stop_l80_s8", "bounded", 80, 8, 64, 3, 1 << 26, slower=26, cap_lo=4.2, cap_hi=12.8),
        _case("early_stop_l126_s16", "bounded", 126, 16, 128, 4, 1 << 24, types="fixed", cap_lo=4.0, cap_hi=16.2),
        # the pruned search over every placement and composition of the 8-stage model
        _case("search_l80_s8", "search", 80, 8, 64, 3, 0, slower=26, cap_lo=4.2, cap_hi=12.8, chunk=512),
    ]


def _spread(rng, lo, hi):
    """A whole number in [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    while True:
        call = rng.choice(["eval"] * 5 + ["noalloc"] * 2 + ["bounded"] * 2 + ["search"])
        T = rng.randint(2, 6)
        if call == "search":
            S = rng.randint(3, 6)
            L = rng.randint(2 * S, 40)
            sched, V, types = rng.choice(["1f1b", "eager"]), 1, "digits"
            T = min(T, 3)
        else:
            S = rng.randint(2, 16)
            L = _spread(rng, S + rng.randint(0, 20), 200)
            sched, V = rng.choice(["1f1b"] * 3 + ["eager", "interleaved"]), 1
            types = rng.choice(["fixed", "table", "digits"])
            if sched == "interleaved":
                V = rng.choice([2, 3, 4])
                if call == "bounded" or S % V or S // V < 2:
                    continue
        M = _spread(rng, 2, 192)
        N = S // V
        if sched == "interleaved":
            M = N * max(1, M // N)
        rows = rng.randint(2, 300) if types == "table" else 0
        A = {"fixed": 1, "table": rows, "digits": T ** N}[types]
        total = math.comb(L - 1, S - 1) * A
        if A >= 1 << 31 or total >= 1 << 62:
            continue
        count = min(_spread(rng, 100, 1 << 22), (1 << 31) // (2 * S * M))
        mode = rng.choice(["list", "range"])
        if mode == "range" or call == "search":
            count = min(count, total)
        if call == "bounded" and mode == "range" and count < WARM:
            continue
        return _case(None, call, L, S, M, T, count, sched, V, types, rows, mode, allreduce=rng.random() < 0.25,
                     slower=rng.randint(12, 30), cap_lo=rng.uniform(2.0, 4.0), cap_hi=rng.uniform(4.5, 14.0),
                     ridge=call == "search" and rng.random() < 0.3,
                     chunk=rng.choice([8, 64, 512]) if call == "search" else 0)


def _problem(case, seed):
    """Profile tables of a case (host arrays), from the seed."""
    rng = np.random.Generator(np.random.PCG64([seed, case["L"], case["S"], case["M"], case["T"]]))
    L, S, M, T, V = (case[k] for k in ("L", "S", "M", "T", "V"))
    N = S // V
    base = np.maximum(np.floor(rng.lognormal(math.log(1000.0), 0.1, size=L) + 0.5), 1)
    base[0] = np.floor(1.5 * base[0])      # the embedding and the head weigh more than a layer
    base[-1] = 2 * base[-1]
    ratio = 1 + (case["slower"] / 10 - 1) * np.arange(T) / max(T - 1, 1)
    fwd = np.floor(base[None, :] * ratio[:, None] + 0.5)
    comm = rng.integers(30, 161, size=S - 1)
    mem = rng.integers(1024, 2049, size=L)
    # caps in units of a device's mean footprint, larger on the slower types
    cap = 1536.0 * L / N * (case["cap_lo"] + (case["cap_hi"] - case["cap_lo"]) * np.arange(T) / max(T - 1, 1))
    if case["types"] == "fixed":
        assign = rng.permutation(np.arange(N) % T).astype(np.uint8)[None, :]
    elif case["types"] == "table":
        assign = rng.integers(0, T, size=(case["rows"], N)).astype(np.uint8)
    else:
        assign = None
    ar = np.floor(rng.integers(20000, 60001, size=L)[None, :] * ratio[:, None]) if case["allreduce"] else None
    u32 = lambda a: np.ascontiguousarray(np.asarray(a, dtype=np.int64).astype(np.uint32))
    return Problem(L, S, M, T, u32(fwd), u32(2 * fwd), u32(comm), u32(comm), u32(mem), u32(cap), assign, seed,
                   None if ar is None else u32(ar), SCHED[case["sched"]], V)


def _lists(case, prob, seed, n):
    """n sampled (composition rank, assignment) pairs on the GPU; the assignments are None when there is one."""
    g = torch.Generator(device="cuda").manual_seed(seed * 1000003 + n)
    ranks = torch.randint(0, prob.n_compositions, (n,), generator=g, device="cuda", dtype=torch.int64)
    rows = torch.randint(0, prob.A, (n,), generator=g, device="cuda", dtype=torch.int32) if prob.A > 1 else None
    return dict(comp_rank=ranks, assign_idx=rows)


def _cands(case, prob, seed):
    if case["mode"] == "range":
        n = case["count"]
        return dict(first=(prob.n_candidates - n) // 3, count=n)
    return _lists(case, prob, seed, case["count"])


def prepare(case, seed):
    prob = _problem(case, seed)
    st = dict(call=case["call"], ctx=P.poseidon_load_costs(prob, 0), ridge=case["ridge"], chunk=case["chunk"])
    if case["call"] != "search":
        st["cands"] = _cands(case, prob, seed)
    if case["call"] in ("search", "bounded"):
        st["warm"] = _lists(case, prob, seed + 7, WARM)
    if case["call"] in ("eval", "noalloc"):
        n = case["count"]
        st["makespan"] = torch.empty(n, dtype=torch.int32, device="cuda")
        st["bits"] = torch.empty((n + 31) // 32, dtype=torch.int32, device="cuda")
    return st


def _best(b):
    return [-1, -1] if b.index is None else [b.index, b.makespan]


def run(st):
    stream = torch.cuda.current_stream()
    if st["call"] in ("eval", "noalloc"):
        f = P.poseidon_eval_candidates if st["call"] == "eval" else P.poseidon_eval_candidates_noalloc
        b = f(st["ctx"], makespan_out=st["makespan"], feasible_bits_out=st["bits"], stream=stream, **st["cands"])
        return {"makespan": st["makespan"], "bits": st["bits"], "best": _best(b)}
    # warm-up: the best of a few hundred samples bounds what follows
    w = P.poseidon_eval_candidates(st["ctx"], stream=stream, **st["warm"])
    bound = 2 ** 31 - 1 if w.makespan is None else w.makespan
    if st["call"] == "bounded":
        b, s = P.poseidon_eval_candidates_bounded(st["ctx"], bound, stream=stream, **st["cands"])
        return {"best": _best(b), "stats": [s.evaluated, s.pruned, s.infeasible]}
    b, s = P.poseidon_search(st["ctx"], bound, rows_per_chunk=st["chunk"], ridge=st["ridge"], ramp=True, stream=stream)
    return {"best": _best(b),
            "stats": [s.visited, s.evaluated, s.pruned_memory, s.pruned_ridge, s.pruned_bound]}


def work(case):
    S, n = case["S"], case["count"]
    listed_in = 8 + (4 if case["types"] != "fixed" else 0) if case["mode"] == "list" else 0
    if case["call"] in ("eval", "noalloc"):
        # per stage two sums, one memory test, the forward and backward legs of a path; one word and a bit out
        return {"bytes": n * (listed_in + 4 + 0.125), "flops": n * 6 * S}
    if case["call"] == "bounded":
        return {"bytes": n * listed_in, "flops": n * 6}          # one stage's two tests decide a candidate
    rows = case["T"] ** case["S"]
    return {"bytes": rows, "flops": rows * 6 * case["L"]}        # the first stage's choices of every placement


def tolerance(case):
    return "exact"


# ---------------------------------------------------------------------------
# The model in plain 64-bit numpy: unrank, sum the stages, walk the DAG node by node.
# ---------------------------------------------------------------------------
def _orders(S, M, sched, V):
    """Per device the nodes ('F' | 'B', virtual stage, micro-batch) in execution order (all 0-based)."""
    out = []
    N = S // V
    for p in range(N):
        if sched == "interleaved":
            F = [("F", (k % S) // N * N + p, k // S * N + k % N) for k in range(V * M)]
            B = [("B", (V - 1 - (k % S) // N) * N + p, k // S * N + k % N) for k in range(V * M)]
            w = V * M if M == N else min(2 * (N - p - 1) + (V - 1) * N, V * M)
        else:
            F = [("F", p, m) for m in range(M)]
            B = [("B", p, m) for m in range(M)]
            w = min(S - p, M) if sched == "1f1b" else min(2 * (S - p) - 1, M)
        o = F[:w]
        for i in range(len(F) - w):
            o += [B[i], F[w + i]] if sched == "eager" else [F[w + i], B[i]] if sched == "interleaved" else [B[i], F[w + i]]
        out.append(o + B[len(F) - w:])
    return out


def _unrank(rank, L, S):
    """Cut points [S+1] of the compositions with these lexicographic ranks."""
    cuts = [np.zeros_like(rank)]
    lo, r = np.zeros_like(rank), rank.copy()
    for k in range(S - 1, 0, -1):           # k cuts left, each above lo
        c, open_ = lo + 1, np.ones(len(r), bool)
        table = np.array([math.comb(n, k - 1) for n in range(L)], dtype=np.int64)
        while open_.any():                  # cut = c leaves C(L-1-c, k-1) compositions
            t = table[np.clip(L - 1 - c, 0, L - 1)]
            open_ &= r >= t
            r = np.where(open_, r - t, r)
            c = np.where(open_, c + 1, c)
        cuts.append(c)
        lo = c
    return cuts + [np.full_like(rank, L)]


def _evaluate(case, prob, rank, row):
    """Makespan and feasibility of these (composition rank, assignment row) pairs."""
    L, S, M, T, V = prob.L, prob.S, prob.M, prob.T, prob.V
    N = S // V
    cuts = _unrank(rank, L, S)
    if prob.assign is not None:
        ty = [prob.assign[:, d].astype(np.int64)[row] for d in range(N)]
    else:
        ty = [row // T ** (N - 1 - d) % T for d in range(N)]
    pre = lambda a: np.concatenate([np.zeros((a.shape[0], 1), np.int64), np.cumsum(a.astype(np.int64), 1)], 1)
    stage = lambda pf, s: pf[ty[s % N], cuts[s + 1]] - pf[ty[s % N], cuts[s]]
    pf, pb, pm = pre(prob.fwd), pre(prob.bwd), pre(prob.mem[None, :])[0]
    W = {("F", s): stage(pf, s) for s in range(S)}
    W.update({("B", s): stage(pb, s) for s in range(S)})
    feas = np.ones(len(rank), bool)
    for d in range(N):
        feas &= sum(pm[cuts[s + 1]] - pm[cuts[s]] for s in range(d, S, N)) <= prob.cap.astype(np.int64)[ty[d]]
    fin, last, at = {}, [0] * N, [0] * N
    orders = _orders(S, M, case["sched"], V)
    left = sum(len(o) for o in orders)
    while left:
        for d in range(N):
            while at[d] < len(orders[d]):
                k, s, m = node = orders[d][at[d]]
                if k == "F":
                    need, edge = (("F", s - 1, m), int(prob.comm_fwd[s - 1])) if s else (None, 0)
                else:
                    need, edge = (("B", s + 1, m), int(prob.comm_bwd[s])) if s < S - 1 else (("F", s, m), 0)
                if need is not None and need not in fin:
                    break
                start = last[d] if need is None else np.maximum(last[d], fin[need] + edge)
                last[d] = fin[node] = W[(k, s)] + start
                if need is not None and (k == "F" or s < S - 1):
                    del fin[need]                      # its other reader is its own device's next node (last)
                at[d] += 1
                left -= 1
    if prob.allreduce is None:
        return last[0], feas
    pd = pre(prob.allreduce)
    return np.max([last[d] + sum(stage(pd, s) for s in range(d, S, N)) for d in range(N)], axis=0), feas


def _argmin(T, feas, base, bound=None):
    key = np.where(feas, T, np.int64(1) << 40)
    i = int(np.argmin(key))
    if not feas[i] or (bound is not None and T[i] > bound):
        return [-1, -1]
    return [base + i, int(T[i])]


def _exact_cands(case, prob, c):
    if "comp_rank" in c:
        rank = c["comp_rank"].cpu().numpy().astype(np.int64)
        row = c["assign_idx"].cpu().numpy().astype(np.int64) if c["assign_idx"] is not None else np.zeros_like(rank)
        return rank, row, 0
    i = np.arange(c["count"], dtype=np.int64) + c["first"]
    return i // prob.A, i % prob.A, c["first"]


def exact(case, seed):
    prob = _problem(case, seed)
    nodes = 2 * case["S"] * case["M"] + 40 * case["S"]
    n = prob.n_candidates if case["call"] == "search" else case["count"] + WARM
    if n * nodes > 1 << 30:
        return None
    if case["call"] in ("bounded", "search"):
        r, a, _ = _exact_cands(case, prob, _lists(case, prob, seed + 7, WARM))
        w = _argmin(*_evaluate(case, prob, r, a), 0)
        bound = 2 ** 31 - 1 if w[0] < 0 else w[1]
    if case["call"] == "search":
        if case["ridge"]:
            return None
        i = np.arange(n, dtype=np.int64)               # search order: assignment row first
        r, a = i % prob.n_compositions, i // prob.n_compositions
        b = _argmin(*_evaluate(case, prob, r, a), 0, bound)
        if b[0] >= 0:
            b[0] = int(r[b[0]]) * prob.A + int(a[b[0]])
        return {"best": b, "stats": [None] * 5}
    r, a, base = _exact_cands(case, prob, _cands(case, prob, seed))
    T, feas = _evaluate(case, prob, r, a)
    if case["call"] == "bounded":
        return {"best": _argmin(T, feas, base, bound), "stats": [None] * 3}
    bits = np.zeros(((len(T) + 31) // 32) * 32, np.uint32)
    bits[:len(T)] = feas
    words = (bits.reshape(-1, 32) << np.arange(32, dtype=np.uint32)).sum(1, dtype=np.uint64).astype(np.uint32)
    return {"makespan": T, "bits": words.view(np.int32).astype(np.int64), "best": _argmin(T, feas, base)}
