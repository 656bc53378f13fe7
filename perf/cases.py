"""Performance cases of the plan-space estimator, the proxy planner and the
scheduling step: what a cluster scheduler calls once per event or per round.

`listed()` names the cases that are reported, `draw()` gives more of the same
ranges, `prepare()` what a caller holds before the call (tables resident on the
GPU, a bound estimator or scheduler), `run()` one pass through the public entry
points, `work()` the bytes and operations a pass cannot do without,
`tolerance()` how far two correct implementations may be apart, and `exact()`
the same outputs from a plain float64 evaluation of the model where that is
quick.  The job, grid and throughput distributions are those of the workload
recipes of this repository (workloads.py, sched_states.py), drawn here for
whole arrays at once.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2403_16125_amd import arena, workloads

# GPU types of the scheduling rounds: speed, GB, GB/s inside a node, GB/s across nodes, node size
TYPES = [(1.0, 96, 300, 25, 8), (0.85, 80, 300, 25, 16), (0.7, 80, 300, 12.5, 4), (0.55, 48, 32, 25, 2),
         (0.45, 40, 300, 12.5, 2), (0.35, 48, 32, 25, 16), (0.25, 24, 32, 12.5, 8), (0.15, 32, 300, 12.5, 4)]
RULES = {"balanced": arena.PARTITION_BALANCED, "memory": arena.PARTITION_MEMORY,
         "exact-t": arena.PARTITION_EXACT_T}


def listed():
    est = dict(call="estimate", rule="balanced", tables=False, cuts=False, shared_kappa=False, mmax=64)
    return [
        # the smallest useful call: a handful of short jobs on a small cluster, with their cuts
        dict(est, name="tiny", kind="uniform", jobs=4, layers=12, batch=32, types=2, counts="pow2", top=8,
             cuts=True, shared_kappa=True, mmax=8),
        # a job arrives: its profile is bound and every (type, count) of the cluster is estimated for it
        dict(est, name="arrival", call="arrival", kind="mixed", jobs=2, layers=0, batch=0, types=8,
             counts="eights", top=1024, cuts=True),
        # a small cluster's queue, odd layer counts, one contention factor per type
        dict(est, name="small", kind="lognormal", jobs=64, layers=0, batch=0, types=3, counts="pow2", top=64,
             cuts=True, shared_kappa=True, mmax=32),
        # a round over a trace-like queue
        dict(est, name="trace", kind="trace", jobs=1024, layers=0, batch=0, types=4, counts="eights", top=256),
        # deep mixture-of-experts jobs, powers of two only, with their cuts
        dict(est, name="moe", kind="moe", jobs=4096, layers=128, batch=0, types=6, counts="pow2", top=512,
             cuts=True, shared_kappa=True),
        # the full scheduling round
        dict(est, name="full round", kind="mixed", jobs=16384, layers=0, batch=0, types=8, counts="eights",
             top=1024),
        # the same round under the memory-constrained partition, an eighth of the jobs, with their cuts
        dict(est, name="memory rule", kind="mixed", jobs=2048, layers=0, batch=0, types=8, counts="eights",
             top=1024, rule="memory", cuts=True),
        # each plan on its split of least iteration time (at most 96 layers)
        dict(est, name="exact-T", kind="trace", jobs=512, layers=0, batch=0, types=4, counts="eights", top=256,
             rule="exact-t"),
        # profiled communication tables
        dict(est, name="comm tables", kind="mixed", jobs=1024, layers=0, batch=0, types=8, counts="eights",
             top=1024, tables=True),
        # the paper's proxy planner over a part of a trace-like queue
        dict(name="proxy", call="proxy", kind="trace", jobs=96, layers=0, batch=0, types=4, counts="eights",
             top=256, n_ops=16, shared_kappa=False, mmax=64),
        # one scheduling step over the full round's matrix
        dict(name="schedule", call="schedule", jobs=16384, types=8, counts="eights", top=1024, per_type=160,
             running=0.5, queued=0.02, classes=3, depth=3, max_count=32, objective="throughput",
             deadlines=False),
        # a step with many small running jobs, finish-time fairness and deadlines
        dict(name="schedule fair", call="schedule", jobs=1500, types=5, counts="pow2", top=128, per_type=600,
             running=0.6, queued=0.1, classes=4, depth=16, max_count=16, objective="fairness",
             deadlines=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["estimate", "estimate", "estimate", "arrival", "proxy", "schedule"])
    types = rng.randint(1, 8)
    counts = rng.choice(["pow2", "eights", "odd"])
    if call == "schedule":
        top = rng.choice([16, 64, 256, 1024])
        return dict(call=call, jobs=_log(rng, 60, 16384), types=types, counts=counts, top=top,
                    per_type=_log(rng, 16, 640), running=round(rng.uniform(0.1, 0.8), 3),
                    queued=round(rng.uniform(0.01, 0.1), 3), classes=rng.randint(1, 4),
                    depth=rng.choice([1, 2, 3, 8, 16]), max_count=rng.choice([4, 16, 32, 64]),
                    objective=rng.choice(["throughput", "fairness"]), deadlines=rng.random() < 0.5)
    kind = rng.choice(["uniform", "lognormal", "trace", "moe", "mixed"])
    layers = rng.randint(1, 128) if kind in ("uniform", "lognormal") else 0
    batch = rng.choice([0, 0, 0, 96, 120, 192, 640])
    common = dict(kind=kind, layers=layers, batch=batch, types=types, counts=counts,
                  shared_kappa=rng.random() < 0.4, mmax=rng.choice([8, 32, 64]))
    if call == "proxy":
        return dict(common, call=call, jobs=_log(rng, 1, 64), top=rng.choice([16, 64, 256]),
                    n_ops=rng.choice([4, 9, 12, 16]))
    if call == "arrival":
        return dict(common, call=call, jobs=_log(rng, 1, 16), top=rng.choice([64, 256, 1024]), rule="balanced",
                    tables=False, cuts=rng.random() < 0.5)
    rule = rng.choice(["balanced", "balanced", "memory", "exact-t"])
    tables = rule == "balanced" and rng.random() < 0.3
    top = rng.choice([8, 64, 256, 1024])
    if rule == "exact-t":
        common["kind"], common["layers"] = rng.choice([("trace", 0), ("uniform", rng.randint(1, 96))])
        top = min(top, 256)
    jobs = _log(rng, 1, 256 if rule == "exact-t" else 512 if tables or rule == "memory" else 4096)
    return dict(common, call=call, jobs=jobs, top=top, rule=rule, tables=tables, cuts=rng.random() < 0.5)


# ------------------------------------------------------------ inputs

def _counts(kind, top):
    if kind == "pow2":
        return [1 << k for k in range(top.bit_length()) if 1 << k <= top]
    if kind == "eights":
        return [1, 2, 4] + list(range(8, top + 1, 8))
    step = max(1, top // 48)
    return sorted({1, 2, 3, 5, 6, 7} | set(range(9, top + 1, step)))


def _jobs(rng, case):
    """Per-layer arrays (f64, concatenated), layer offsets and batches of the case's jobs."""
    n, kind = case["jobs"], case["kind"]
    if kind == "mixed":
        moe = rng.random(n) >= 0.7
    else:
        moe = np.full(n, kind == "moe")
    simple = kind in ("uniform", "lognormal")
    if simple:
        L = np.full(n, case["layers"]) if case["layers"] else rng.integers(12, 49, n)
        batch = rng.choice([64, 128, 256], n)
    else:
        L = np.where(moe, 128, rng.integers(24, 97, n))
        batch = np.where(moe, rng.choice([256, 512, 1024], n), rng.choice([128, 256, 512], n))
    if case["batch"]:
        batch = np.full(n, case["batch"])
    off = np.concatenate([[0], np.cumsum(L)])
    job = np.repeat(np.arange(n), L)
    total = int(off[-1])
    if simple:
        t = rng.uniform(1e-3, 5e-3, total) if kind == "uniform" else np.exp(math.log(3e-3) + 0.5 * rng.normal(size=total))
        p, a = rng.uniform(50e6, 150e6, total), rng.uniform(20e6, 60e6, total)
        return t, p, a, a / 16.0, np.zeros(total), off, batch
    seq, f_ref = workloads.SEQ_LEN, workloads.F_REF
    lo, hi = math.log(3e8), math.log(7e10)
    pi = np.exp(np.clip((lo + hi) / 2 + (hi - lo) / 4 * rng.normal(size=n), lo, hi)) / L   # parameters of a layer
    h = np.where(moe, rng.choice([1024, 2048, 4096], n), 64 * np.maximum(1, np.round(np.sqrt(pi / 12.0) / 64.0)))
    pi = np.where(moe, 12.0 * h * h, pi)
    odd = ((np.arange(total) - off[job]) % 2 == 1) & moe[job]      # a mixture-of-experts layer
    mul = np.where(odd, 3.0, 1.0)
    noise = np.where(moe[job], np.exp(0.8 * rng.normal(size=total)), 1.0 + rng.uniform(-0.2, 0.2, total))
    t = (6.0 * pi * batch * seq / f_ref)[job] * noise * mul
    a1 = (64.0 * seq * h)[job]
    return t, 4.0 * pi[job] * mul, a1 * mul, a1 / 16.0, np.where(odd, (seq * h * 2.0)[job], 0.0), off, batch


def _workload(case, seed):
    rng = np.random.default_rng([240316125, int(seed)])
    t, p, a, x, q, off, batch = _jobs(rng, case)
    counts = _counts(case["counts"], case["top"])
    ty = np.asarray(TYPES[: case["types"]], np.float64)
    grids = len(ty) * len(counts)
    kappa = (np.ones(grids) if case["shared_kappa"] else rng.uniform(1.0, 2.0, grids)).astype(np.float32)
    f = lambda v: np.ascontiguousarray(v, np.float32)
    return workloads.Workload(
        name="case", seed=int(seed), layer_offset=off.astype(np.int32), t=f(t), p=f(p), a=f(a), x=f(x), a2a=f(q),
        batch=batch.astype(np.int32), speed=f(ty[:, 0]), mem=f(ty[:, 1] * 1e9), bw_intra=f(ty[:, 2] * 1e9),
        bw_inter=f(ty[:, 3] * 1e9), gpus_per_node=ty[:, 4].astype(np.int32), counts=np.asarray(counts, np.int32),
        m_values=np.asarray([1 << k for k in range(7) if 1 << k <= case["mmax"]], np.int32), kappa=kappa[None])


def _sched_state(case, seed):
    """Throughput curves (zero below a job's smallest count, then growing with diminishing
    returns, faster on faster types) and a cluster state over them."""
    rng = np.random.default_rng([24031612, int(seed)])
    J, T = case["jobs"], case["types"]
    counts = np.asarray(_counts(case["counts"], case["top"]), np.int64)
    NC = len(counts)
    dev = torch.device("cuda")
    gen = lambda v: torch.as_tensor(np.ascontiguousarray(v), device=dev)
    speed = np.sort(rng.uniform(0.2, 1.0, T))[::-1]
    alpha = rng.uniform(0.45, 0.95, J)
    base = np.exp(rng.uniform(math.log(5.0), math.log(500.0), J))
    nmin = rng.choice(counts[: max(1, NC // 2)], J)
    least = np.maximum(1, np.ceil(nmin[:, None] / np.sqrt(speed)[None, :]))
    c = gen(counts.astype(np.float64))
    curve = gen(base)[:, None, None] * gen(speed.copy())[None, :, None] * c[None, None, :] ** gen(alpha)[:, None, None]
    thr = torch.where(c[None, None, :] >= gen(least)[:, :, None], curve, torch.zeros_like(curve)).float().contiguous()
    # running jobs in random order on a random open grid of at most max_count GPUs, while it fits
    at, ac = np.full(J, -1, np.int32), np.zeros(J, np.int32)
    u = rng.random(J)
    pick_g, pick = rng.integers(0, T, J), rng.random(J)
    left = np.full(T, case["per_type"], np.int64)
    for j in np.nonzero(u < case["running"])[0]:
        g = int(pick_g[j])
        lo = int(np.searchsorted(counts, least[j, g]))
        hi = int(np.searchsorted(counts, min(case["max_count"], int(left[g])), side="right"))
        if lo < hi:
            k = lo + int(pick[j] * (hi - lo))
            at[j], ac[j] = g, k
            left[g] -= counts[k]
        if left.max() <= 0:
            break
    # a share of the jobs that were not drawn as running waits in the queue
    nq = max(1, int(case["queued"] * J))
    idle = np.nonzero(u >= case["running"])[0]
    idle = np.concatenate([idle, np.setdiff1d(np.nonzero(at < 0)[0], idle)])[:nq]
    queue = np.sort(idle)
    prio = np.sort(rng.integers(0, case["classes"], len(queue)))
    batch = rng.choice([64, 128, 256, 512], J).astype(np.int32)
    iters = np.exp(rng.uniform(math.log(1e3), math.log(1e5), J)).astype(np.float32)
    best = (base * speed[0] * float(counts[-1]) ** alpha)
    ddl = np.where(rng.random(J) < 0.3, np.inf, batch * iters.astype(np.float64) / best * rng.uniform(0.8, 6.0, J))
    return thr, counts.astype(np.int32), at, ac, queue.astype(np.int32), prio.astype(np.int32), batch, iters, ddl.astype(np.float32)


def prepare(case, seed):
    if case["call"] == "schedule":
        thr, counts, at, ac, queue, prio, batch, iters, ddl = _sched_state(case, seed)
        fair = case["objective"] == "fairness"
        assert len(queue) == max(1, int(case["queued"] * case["jobs"]))
        s = arena.Scheduler(thr, counts, [case["per_type"]] * case["types"], objective=case["objective"])
        if fair or case["deadlines"]:
            s.set_deadlines(batch, iters, ddl if case["deadlines"] else None)
        s.load_state(at, ac, queue, prio)
        return dict(case=case, s=s, at=s.alloc_type.clone(), ac=s.alloc_count.clone())
    w = _workload(case, seed)
    est = arena.Estimator(w, with_cuts=case.get("cuts", False), rule=RULES[case.get("rule", "balanced")],
                          comm_tables=workloads.comm_tables(w) if case.get("tables") else None)
    if case["call"] == "proxy":      # the proxy planner's output buffers are made once by its first call
        c = est.n_cells
        est.p_t_iter, est.p_thr = est.t_iter, est.thr
        est.p_plan = torch.empty(c * 3, dtype=torch.int64, device=est.dev)
    return dict(case=case, est=est, w=w, kappa=w.kappa[0], hbm=w.hbm_bw())


def run(state):
    call = state["case"]["call"]
    if call == "schedule":
        s = state["s"]
        # the cluster state of this event, then the step
        s.alloc_type.copy_(state["at"])
        s.alloc_count.copy_(state["ac"])
        s.step(state["case"]["depth"])
        return {"alloc_type": s.alloc_type, "alloc_count": s.alloc_count, "launched": s.launched[: s.n_queue],
                "result": s.result}
    est = state["est"]
    if call == "proxy":
        est.proxy_estimate(f_ref=workloads.F_REF, n_ops=state["case"]["n_ops"], hbm_bw=state["hbm"])
        return {"t_iter": est.p_t_iter, "thr": est.p_thr, "plan": est.p_plan}
    if call == "arrival":
        w = state["w"]
        arena.arena_bind_jobs(est.ctx, w.layer_offset, w.batch, est.t, est.p, est.a, est.x, est.a2a)
    else:
        est.set_kappa(state["kappa"])        # the contention factors of this round
    est.estimate()
    out = {"t_iter": est.t_iter, "thr": est.thr, "plan": est.plan}
    if est.cuts is not None:
        out["cuts"] = est.cuts
    return out


# ------------------------------------------------------------ what a pass cannot do without

def work(case):
    nc = len(_counts(case["counts"], case["top"]))
    J, T = case["jobs"], case["types"]
    if case["call"] == "schedule":
        # the queued jobs' rows and the allocation in and out; a launch and a scale-down search per queued job
        queue = case["queued"] * J
        return {"bytes": queue * T * nc * 4 + 16.0 * J + 12 * queue, "flops": queue * T * nc}
    L = case["layers"] or {"uniform": 30, "lognormal": 30, "trace": 60, "moe": 128, "mixed": 80}[case["kind"]]
    cells = J * T * nc
    if case["call"] == "proxy":
        # one bias term set and one memory test per stage of every contiguous grouping of the operators
        o = min(L, case["n_ops"])
        stages = sum(math.comb(o - 1, s - 1) * s for s in range(1, o + 1))
        return {"bytes": J * L * 20 + cells * 32, "flops": cells * stages * 11}
    # every cell's best plan built and priced once: layer costs and prefix, the split's test, the sums
    flops = cells * (16.0 * L + 100)
    return {"bytes": J * L * 20 + cells * (12.0 + (arena.CUTS_STRIDE if case["cuts"] else 0)), "flops": flops}


def tolerance(case):
    if case["call"] == "schedule":
        return "exact"
    # times are float64 sums rounded once to float32 (6e-8): a few of those roundings.  Plans, cuts and
    # proxy words are whole numbers; a plan may differ where two iteration times meet the tie window
    # within the last bit of a sum.
    return {"rel": 2.5e-7, "max": 5e-7, "differ": 1e-6}


# ------------------------------------------------------------ float64 reference

def _split(U, pp, fits):
    """The balanced split of prefix U into pp stages among those whose stage k over [i, e) fits
    (fits[k][i, e]; None: all): the least largest stage, then the lexicographically smallest cuts."""
    L = len(U) - 1
    seg = U[None, :] - U[:, None]                       # [i, e]
    seg = np.where(np.arange(L + 1)[:, None] < np.arange(L + 1)[None, :], seg, np.inf)
    ok = lambda k: seg if fits is None else np.where(fits[k], seg, np.inf)
    G = [np.where(np.arange(L + 1) == L, 0.0, np.inf)]  # G[t][i]: t stages cover [i, L)
    for t in range(1, pp + 1):
        G.append(np.min(np.maximum(ok(pp - t), G[-1][None, :]), axis=1))
    W = G[pp][0]
    if not np.isfinite(W):
        return None, None
    cuts, at = [0], 0
    for k in range(pp - 1):
        e = np.nonzero((ok(k)[at] <= W) & (G[pp - k - 1] <= W))[0][0]
        cuts.append(int(e))
        at = int(e)
    return W, np.asarray(cuts + [L])


def _latency(v, vol, lat):
    v = np.asarray(v, np.float64)
    k = np.clip(np.searchsorted(vol, v, side="right") - 1, 0, len(vol) - 2)
    f = lat[k] + (v - vol[k]) * ((lat[k + 1] - lat[k]) / (vol[k + 1] - vol[k]))
    return np.where(v > 0, f, 0.0)


def exact(case, seed):
    """t_iter and thr of every cell in float64; plans and cuts are whole numbers, without such a value.
    Not for the searches that plain loops cannot do in seconds: larger workloads, the exact-T split
    and the proxy planner's groupings."""
    if case["call"] not in ("estimate", "arrival") or case["rule"] == "exact-t":
        return None
    nc = len(_counts(case["counts"], case["top"]))
    most = 150 if case["tables"] or case["rule"] == "memory" else 1500
    if case["jobs"] * case["types"] * nc > most or case["kind"] in ("moe", "mixed"):
        return None
    w = _workload(case, seed)
    tabs = workloads.comm_tables(w) if case["tables"] else None
    T_out = np.full((w.n_jobs, w.n_types, w.n_counts), np.inf)
    for j in range(w.n_jobs):
        s = w.job_slice(j)
        t, p, a, x, q = (getattr(w, k)[s].astype(np.float64) for k in ("t", "p", "a", "x", "a2a"))
        L, Bg = len(t), int(w.batch[j])
        cp, ca = (np.concatenate([[0.0], np.cumsum(v)]) for v in (p, a))
        for g in range(w.n_types):
            node, mem, speed = int(w.gpus_per_node[g]), float(w.mem[g]), float(w.speed[g])
            bw = (float(w.bw_intra[g]), float(w.bw_inter[g]))
            cost = lambda link, v: v / bw[link] if tabs is None else _latency(v, tabs[0][g, link], tabs[1][g, link])
            for c in range(w.n_counts):
                n, kap = int(w.counts[c]), float(w.kappa[0][g * w.n_counts + c])
                plans, splits = [], {}
                for tp in (d for d in range(1, node + 1) if node % d == 0 and n % d == 0):
                    for pp in (d for d in range(1, min(L, n // tp) + 1) if (n // tp) % d == 0):
                        dp = n // (tp * pp)
                        for m in (int(v) for v in w.m_values if Bg % (dp * int(v)) == 0):
                            b = Bg // (dp * m)
                            on = dp * tp > 1
                            # per-microbatch layer costs
                            u = t * b / (Bg * speed * tp)
                            if tp > 1:
                                u = u + kap * 4 * cost(0, 2 * (tp - 1) / tp * b * x)
                            if on:
                                u = u + kap * cost(1, b * q)
                            inflight = np.minimum(m, pp - np.arange(pp))
                            stage_mem = lambda k, P, A: 4 * P / tp + inflight[k] * b * A / tp
                            key = (tp, on, pp) if tabs is None else (tp, on, pp, b)
                            if key not in splits:
                                _, cuts = _split(np.concatenate([[0.0], np.cumsum(u / b)]), pp, None)
                                splits[key] = cuts
                            cuts = splits[key]
                            P, A = np.diff(cp[cuts]), np.diff(ca[cuts])
                            if not (stage_mem(np.arange(pp), P, A) <= mem).all():
                                if case["rule"] != "memory":
                                    continue
                                dP, dA = cp[None, :] - cp[:, None], ca[None, :] - ca[:, None]
                                _, cuts = _split(np.concatenate([[0.0], np.cumsum(u / b)]), pp,
                                                 [stage_mem(k, dP, dA) <= mem for k in range(pp)])
                                if cuts is None:
                                    continue
                                P = np.diff(cp[cuts])
                            S = np.add.reduceat(u, cuts[:-1])
                            pl = 0 if n <= node else 1
                            dl = 0 if node % (dp * tp) == 0 else 1
                            p2p = kap * 2 * np.sum(cost(pl, b * x[cuts[1:-1] - 1])) if pp > 1 else 0.0
                            ar = kap * cost(dl, 2 * (dp - 1) / dp * np.max(P) / tp) if dp > 1 else 0.0
                            plans.append((pp, tp, m, float(np.sum(S) + p2p + (m - 1) * np.max(S) + ar)))
                if plans:
                    top = min(v[3] for v in plans) * (1 + w.tie_eps)
                    T_out[j, g, c] = min(v for v in plans if v[3] <= top)[3]
    T_out = T_out.reshape(-1)
    thr = np.where(np.isfinite(T_out), np.repeat(w.batch.astype(np.float64), w.n_types * w.n_counts) / T_out, 0.0)
    out = {"t_iter": T_out, "thr": thr, "plan": None}
    if case["cuts"]:
        out["cuts"] = None
    return out
