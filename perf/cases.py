"""What is timed: the calls a user of this planner makes, over the range of traces they make them on.

A case is a dict: which call (`call`), which trace (`trace` and, for the synthetic stress family, its sizes), and the
machine it is planned for.  The planner works in whole nanoseconds and bytes on one data type, so every result is
compared exactly.

  call "step"      profile -> plan, the cycle that repeats per trace: analysis of a trace that lies in GPU memory, one
                   eviction plan, the handle given back
  call "plan"      a plan on an analysed trace (re-planning for another machine), in one of the readings of the paper:
                   ranking by benefit (rank 0) or benefit / cost (rank 1), the benefit as the tensor's band (area 0) or
                   as the area above the capacity line (area 1)
  call "batch"     a sensitivity study in one call: `plans` plans of one trace over a range of capacities ("capacity"),
                   flash bandwidths ("bandwidth") or profiling errors of the kernel times ("noise")
  call "follow"    what follows a plan: smart prefetching, and the replay of the plan with and without it, under the
                   profiled and under noisy kernel times
  call "analysis"  the analysis alone, into buffers the caller holds, without an allocation
"""
import math

import numpy as np
import torch

from paper_2310_09443_amd import binding, traces

MODELS = {"mlp": traces.mlp_tiny, "encoder": traces.encoder12, "resnet": traces.resnet152, "decoder": traces.decoder48}
# kernels, tensors, use pairs of the model traces (the seed changes durations and temporaries' sizes, not these)
MODEL_SIZES = {"mlp": (24, 34, 80), "encoder": (1337, 2876, 5273), "resnet": (5849, 15167, 26557), "decoder": (12403, 39524, 65099)}

BASE = {"call": "step", "trace": "stress", "K": 0, "N": 0, "cap": 0.25, "host": 0.25, "flash_MBps": 6000, "host_MBps": 25000,
        "rank": 0, "area": 0, "max_iters": 0, "plans": 1, "sweep": "", "wrap": True}


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a four-layer MLP, 24 kernels; launches and latency are all there is
        _case(name="step_mlp", trace="mlp", cap=0.60),
        # the model traces of the benchmark, each on the machine it names there
        _case(name="step_encoder", trace="encoder", cap=0.50),
        _case(name="step_resnet", trace="resnet", cap=0.40, flash_MBps=12000),
        _case(name="step_decoder", trace="decoder", cap=0.30),
        # the stress trace of the benchmark: 100 000 kernels, 1 000 000 tensors
        _case(name="step_stress", K=100000, N=1000000),
        # a ragged trace between those, weights not kept across iterations, host memory so tight that it refuses candidates
        _case(name="step_ragged", K=20011, N=150007, cap=0.37, host=0.03, flash_MBps=12800, wrap=False),
        # the analysis alone, as large as its fixed memory takes
        _case(name="analysis_static", call="analysis", K=9001, N=90007),
        # the evaluation of a finished plan
        _case(name="follow_stress", call="follow", K=100000, N=1000000),
        # sensitivity studies: capacity on the stress trace, profiling errors on a model trace
        _case(name="batch_capacity", call="batch", K=100000, N=1000000, plans=20, sweep="capacity"),
        _case(name="batch_noise", call="batch", trace="decoder", cap=0.30, plans=6, sweep="noise"),
        # the alternative readings: benefit / cost on the stress trace (its first passes, as the benchmark does) ...
        _case(name="plan_ratio", call="plan", K=100000, N=1000000, rank=1, max_iters=500),
        # ... and the area above the capacity line on a model trace
        _case(name="plan_clipped", call="plan", trace="resnet", cap=0.40, flash_MBps=12000, area=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["step", "step", "step", "plan", "batch", "follow", "analysis"])
    machine = dict(cap=round(rng.uniform(0.2, 0.7), 4), host=rng.choice([0.02, 0.05, 0.25, 0.5]),
                   flash_MBps=rng.randint(6000, 32000), wrap=rng.random() < 0.8)
    if call == "analysis":
        K = _log(rng, 24, 12000)                  # (at most 262144 pairs)
        return _case(call=call, K=K, N=min(_log(rng, 24, 88000), 12 * K), **machine)
    if rng.random() < 0.5:
        size = dict(trace=rng.choice(["mlp", "encoder", "resnet", "decoder"]))
    else:
        K = _log(rng, 24, 100000 if call in ("step", "follow") else 30000)
        size = dict(K=K, N=max(16, min(1000000, int(K * rng.uniform(2.0, 10.0)))))
    kind = dict()
    if call == "plan":                # (the first passes of a plan; clipped areas cost up to 0.7 ms a pass where layers repeat)
        area = rng.choice([0, 1])
        kind = dict(rank=rng.choice([0, 1]), area=area, max_iters=rng.randint(20, 60) if area else rng.randint(100, 600))
    if call == "batch":
        kind = dict(plans=rng.randint(2, 20), sweep=rng.choice(["capacity", "bandwidth", "noise"]))
        if kind["sweep"] == "noise":
            kind["plans"] = min(kind["plans"], 6)
    return _case(call=call, **size, **kind, **machine)


def _workload(case, seed):
    if case["trace"] == "stress":
        w = traces.stress(case["K"], case["N"], seed=0x67100005 + 977 * seed)
    else:
        w = MODELS[case["trace"]](seed=0x67100000 + 977 * seed)
    return w.trace


def _caps(case, peak):
    return peak * int(round(case["cap"] * 10000)) // 10000, peak * int(round(case["host"] * 10000)) // 10000


def _machine(case, peak):
    cap, host = _caps(case, peak)
    bw = (case["flash_MBps"], case["host_MBps"])
    return dict(gpu_cap=cap, host_cap=host, bw_out=bw, bw_in=bw)


def _noise(tr, percent, seed):
    return torch.from_numpy(traces.noisy_durations(tr, percent, seed).view(np.int64)).cuda()


class _Kept:
    """An array for results of varying length: the rows after the last result's are zeros."""

    def __init__(self, rows, dtype, as_numbers):
        self.a, self.n, self.as_numbers = np.zeros(rows, dtype), 0, as_numbers

    def take(self, x):
        n = len(x)
        self.a[:n] = x                            # (raises if it does not fit)
        self.a[n:self.n] = np.zeros((), self.a.dtype)
        self.n = n
        return self.a.view(self.as_numbers)


def prepare(case, seed):
    tr = _workload(case, seed)
    dt = binding.DeviceTrace(tr)
    st = {"case": case, "trace": dt, "no_wrap": not case["wrap"]}
    # the arrays a program keeps for its plans: as long as any plan of such a trace can get, zeros after the plan's end
    rows = min(2 * tr.N, 16384 + tr.N // 32) + 64
    if case["call"] in ("step", "plan", "batch"):
        st["out"] = [{"records": _Kept(rows, binding.MIGRATION, np.int64), "dropped": _Kept(rows, binding.DROPPED, np.int64)}
                     for _ in range(case["plans"])]
    elif case["call"] == "follow":
        st["out"] = {**{n: _Kept(rows, np.dtype("<u4"), np.int32) for n in ("order", "gained", "absent_last")},
                     **{"late_" + n: _Kept(rows, np.dtype("<u8"), np.int64) for n in ("planned", "prefetched", "noisy")}}
    if case["call"] == "step":
        return st
    if case["call"] == "analysis":
        n = lambda k, t: torch.zeros(k, dtype=t, device="cuda")      # noqa: E731
        P = binding.STATIC_MAX_P                  # (room for any trace the call takes)
        st["buffers"] = dict(use_off=n(tr.N + 1, torch.int64), use_k=n(P, torch.int32), per_tensor=n(P, torch.int32),
                             per_L=n(P, torch.int32), per_R=n(P, torch.int32), start=n(tr.K + 1, torch.int64),
                             pressure=n(tr.K, torch.int64))
        return st
    h = binding.g10_vitality(dt, no_wrap=not case["wrap"])
    st["handle"] = h
    m = _machine(case, h.peak)
    if case["call"] == "plan":
        st["params"] = dict(m, rank=case["rank"], area=case["area"], max_iters=case["max_iters"])
    elif case["call"] == "follow":
        h.plan(**m)
        st["noise"] = _noise(tr, 20.0, 2020 + seed)
    else:
        n = case["plans"]
        if case["sweep"] == "capacity":          # from a fifth under to two fifths over the case's capacity
            ps = [dict(m, gpu_cap=int(m["gpu_cap"] * (0.8 + 0.6 * i / (n - 1)))) for i in range(n)]
        elif case["sweep"] == "bandwidth":       # flash from 6.4 to 32 GB/s
            fl = [6400 + (32000 - 6400) * i // (n - 1) for i in range(n)]
            ps = [dict(m, bw_out=(f, case["host_MBps"]), bw_in=(f, case["host_MBps"])) for f in fl]
        else:                                    # profiling errors from 0 to 25 %
            ps = [dict(m, dur=_noise(tr, 25.0 * i / (n - 1), 1000 + i + seed) if i else None) for i in range(n)]
        st["params"] = ps
    return st


def _plan_out(r, out):
    return {"records": out["records"].take(r.records), "dropped": out["dropped"].take(r.dropped), "pressure": r.pressure_after.view(np.int64),
            "counts": np.array([r.status, r.n_iterations, r.n_migrations, r.n_dropped, r.n_cand_evals, r.peak_before, r.peak_after,
                                r.overtime_before_ns, r.overtime_after_ns], np.uint64).view(np.int64)}


def run(state):
    case, call = state["case"], state["case"]["call"]
    if call == "step":
        h = binding.g10_vitality(state["trace"], no_wrap=state["no_wrap"])
        r = h.plan(**_machine(case, h.peak), rank=case["rank"], area=case["area"], max_iters=case["max_iters"])
        n = [h.n_uses, h.C, h.T]
        h.close()
        return dict(_plan_out(r, state["out"][0]), analysis=np.array(n, np.int64))
    if call == "analysis":
        s = binding.g10_vitality_static(state["trace"], no_wrap=state["no_wrap"], buffers=state["buffers"])
        return dict(state["buffers"], counts=np.array([s.n_uses, s.C, s.peak, s.T], np.uint64).view(np.int64))
    h = state["handle"]
    if call == "plan":
        return _plan_out(h.plan(**state["params"]), state["out"][0])
    if call == "batch":
        rs = [_plan_out(r, o) for r, o in zip(h.plan_batch(state["params"]), state["out"])]
        return {"records": [r["records"] for r in rs], "dropped": [r["dropped"] for r in rs], "pressure": [r["pressure"] for r in rs],
                "counts": np.concatenate([r["counts"] for r in rs])}
    pf, keep = h.prefetch(), state["out"]
    out = {"order": keep["order"].take(pf.order), "gained": keep["gained"].take(pf.gained), "absent_last": keep["absent_last"].take(pf.absent_last),
           "pressure": pf.pressure.view(np.int64), "moved": np.array([pf.n_moved, pf.slots_gained, pf.peak], np.uint64).view(np.int64)}
    for name, dur, eager in (("planned", None, False), ("prefetched", None, True), ("noisy", state["noise"], True)):
        rp = h.replay(dur, eager)
        out["late_" + name] = keep["late_" + name].take(rp.late)
        out["replay_" + name] = np.array([rp.iter_ns, rp.planned_ns, rp.stall_ns, rp.n_stalled] + rp.bytes + rp.busy_out_ns + rp.busy_in_ns,
                                         np.uint64).view(np.int64)
    return out


def work(case):
    """Each input read once, each output written once.  (How many migrations a plan makes is only known afterwards:
    about one per hundred tensors of the stress traces; the model traces' plans lie around one per twenty tensors.)"""
    if case["trace"] == "stress":
        K, N = case["K"], case["N"]
        P = int(2.2 * N + 5.05 * K)
        migrations = N // 100
    else:
        K, N, P = MODEL_SIZES[case["trace"]]
        migrations = N // 20
    if case["max_iters"]:
        migrations = min(migrations, case["max_iters"])
    trace = 8 * K + 9 * N + 8 * P
    if case["call"] == "analysis":                # use lists, periods (about half as many as uses), start times, pressure
        return {"bytes": trace + 8 * N + 4 * P + 12 * (P // 2) + 16 * K, "flops": 0}
    if case["call"] == "step":
        return {"bytes": trace + 8 * K + 72 * migrations, "flops": 0}
    periods = P // 2
    if case["call"] == "plan":                    # the periods (tensor, start, end), sizes, durations and pressure in; the plan out
        return {"bytes": 12 * periods + 8 * N + 24 * K + 72 * migrations, "flops": 0}
    if case["call"] == "batch":
        return {"bytes": 12 * periods + 8 * N + 8 * K + case["plans"] * (16 * K + 72 * migrations), "flops": 0}
    # prefetching: plan and pressure in, order, gain and last slot per migration and the pressure out; three replays: the
    # plan and the start times in, the lateness out
    return {"bytes": 72 * migrations + 16 * K + 12 * migrations + 3 * (72 * migrations + 8 * K + 8 * migrations), "flops": 0}


def tolerance(case):
    return "exact"                                # whole numbers throughout


def exact(case, seed):
    """The analysis from its definitions in numpy.  (The plans are a chain of thousands of dependent rankings: minutes of
    numpy for all but the smallest; they are whole numbers and compared as such.)"""
    if case["call"] != "analysis":
        return None
    tr = _workload(case, seed)
    K, N = tr.K, tr.N
    key = np.unique(tr.use_tensor.astype(np.int64) * K + tr.use_kernel.astype(np.int64))
    t, k = key // K, key % K
    use_off = np.searchsorted(t, np.arange(N + 1))
    first, last = use_off[t], use_off[t + 1] - 1
    i = np.arange(len(key))
    inner = (i > first) & (k - np.roll(k, 1) >= 2)
    wrap = (i == last) & (tr.is_global[t] != 0) & (k[first] + K - k >= 2) & case["wrap"]
    cnt = inner.astype(np.int64) + wrap
    pos = np.cumsum(cnt) - cnt
    C = int(cnt.sum())
    per_t, per_L, per_R = (np.zeros(C, np.int64) for _ in range(3))
    per_t[pos[inner]], per_L[pos[inner]], per_R[pos[inner]] = t[inner], np.roll(k, 1)[inner], k[inner]
    at = (pos + inner)[wrap]
    per_t[at], per_L[at], per_R[at] = t[wrap], k[wrap], k[first][wrap] + K
    diff = np.zeros(K + 1, np.int64)
    used = np.flatnonzero(use_off[1:] > use_off[:-1])
    size, glob = tr.size_bytes.view(np.int64), tr.is_global != 0
    birth, death = np.where(glob[used], 0, k[use_off[used]]), np.where(glob[used], K - 1, k[use_off[used + 1] - 1])
    np.add.at(diff, birth, size[used])
    np.add.at(diff, death + 1, -size[used])
    pressure = np.cumsum(diff)[:K]
    start = np.concatenate([[0], np.cumsum(tr.dur_ns.view(np.int64))])
    full = lambda a: np.pad(a, (0, binding.STATIC_MAX_P - len(a))).astype(np.int32)          # noqa: E731
    return {"use_off": use_off, "use_k": full(k), "per_tensor": full(per_t), "per_L": full(per_L), "per_R": full(per_R), "start": start, "pressure": pressure,
            "counts": np.array([len(key), C, pressure.max(), start[-1]], np.int64)}
