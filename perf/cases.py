"""Performance cases of the schedule search: the calls a planner makes, over the sizes it
makes them at.

Every case goes through paper_2601_17654_amd.binding with its default options unless the
case says otherwise, so the input check and the read-back of the result sizes count where
a planner pays for them.  Tables, points and kept output buffers are on the GPU before a
pass, as in a planner's own process.  The kinds:

  plan    partition frontiers of one comm kernel, their composition over time bins, and
          the schedules behind the fastest points of the composed frontier
  eval    evaluation + frontier of every partition (one or two comm kernels), put into the
          planner's own arrays
  points  time and energy of every candidate, then one frontier per (partition,
          frequency): what the microbatch calls take
  compose composition of partition frontiers and the schedule of its fastest point
  mbo     one round of the Bayesian optimisation: scores, uncertainty, batch selection
  grid    microbatch frontier on a time grid
  enum    microbatch frontier by enumeration
  timing  launch-timing frontiers of two operation sequences
"""

import itertools
import math

import numpy as np
import torch

from paper_2601_17654_amd import binding as kr
from paper_2601_17654_amd import inputs as I

P_STATIC = I.P_STATIC_W
QUERIES = 128     # schedules a plan asks for
ENUM_CAP = 65536  # points kept of an enumerated microbatch frontier


def listed():
    return [
        # A first look at a small model: four partitions, everything in microseconds.
        dict(name="plan_tiny", kind="plan", parts=4, kernels=6, comm=1, pos=7, sms=8, freqs=16,
             bins=1024),
        # One transformer model's partitions at the resolution of its frequency grid.
        dict(name="plan_llama", kind="plan", parts=64, kernels=24, comm=1, pos=25, sms=16,
             freqs=64, bins=16384),
        # Two collectives per partition (unfused consecutive ones).
        dict(name="eval_two_comm", kind="eval", parts=256, kernels=48, comm=2, pos=33, sms=8,
             freqs=32, checked=True),
        # The largest batch: 138 million candidates, 2.3 GB of tables.
        dict(name="eval_stress", kind="eval", parts=1024, kernels=32, comm=1, pos=33, sms=32,
             freqs=128, checked=True),
        # Sizes that are no multiples of anything, from a caller that checked its tables.
        dict(name="eval_ragged", kind="eval", parts=301, kernels=41, comm=1, pos=42, sms=19,
             freqs=91, checked=False),
        # The microbatch calls' input for every partition of a model.
        dict(name="points_llama", kind="points", parts=64, kernels=24, comm=1, pos=25, sms=16,
             freqs=64),
        # The iteration frontier of a large model, 512 partitions.
        dict(name="compose_stress", kind="compose", parts=512, lo=256, hi=2048, bins=65536),
        # One optimisation round of a model's partitions.
        dict(name="mbo_llama", kind="mbo", parts=64, kernels=24, comm=1, pos=25, sms=16, freqs=64,
             obs=96, members=5, batch=32),
        # The same over large candidate spaces.
        dict(name="mbo_stress", kind="mbo", parts=128, kernels=32, comm=1, pos=33, sms=32,
             freqs=128, obs=96, members=5, batch=32),
        # A 16-layer microbatch of four partition types.
        dict(name="microbatch_grid", kind="grid", types=4, layers=16, kernels=24, pos=25, sms=16,
             freqs=64, comps=2, bins=4096),
        dict(name="microbatch_enum", kind="enum", types=4, layers=16, kernels=24, pos=25, sms=16,
             freqs=64, comps=2),
        # Launch timing of two nanobatches for every (partition, frequency, SM choice).
        dict(name="launch_timing", kind="timing", parts=256, before=4, after=5, kmax=9, sms=8,
             freqs=32, sched=True),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["plan", "eval", "eval", "points", "compose", "mbo", "grid", "enum",
                       "timing"])
    if kind == "compose":
        lo = _log(rng, 4, 256)
        return dict(kind=kind, parts=_log(rng, 2, 512), lo=lo, hi=_log(rng, lo, 2048),
                    bins=_log(rng, 500, 65536))
    if kind in ("grid", "enum"):
        return dict(kind=kind, types=rng.randint(1, 4), layers=rng.randint(1, 40),
                    kernels=rng.randint(6, 32), pos=rng.randint(3, 7), sms=rng.randint(2, 16),
                    freqs=_log(rng, 4, 128), comps=rng.randint(0, 4),
                    **(dict(bins=_log(rng, 256, 4096)) if kind == "grid" else {}))
    if kind == "timing":
        return dict(kind=kind, parts=_log(rng, 1, 128), before=rng.randint(2, 5),
                    after=rng.randint(2, 5), kmax=rng.randint(2, 9), sms=rng.randint(1, 8),
                    freqs=rng.randint(4, 32), sched=rng.random() < 0.5)
    comm = 2 if kind == "eval" and rng.random() < 0.5 else 1
    kernels = rng.randint(4, 48)
    c = dict(kind=kind, parts=1, kernels=kernels, comm=comm, pos=rng.randint(2, min(kernels + 1, 33)),
             sms=rng.randint(2, 8 if comm == 2 else 32), freqs=_log(rng, 8, 128))
    per = _space(c).n_cand
    most = {"plan": 20e6, "eval": 200e6 if comm == 2 else 60e6, "points": 20e6, "mbo": 12e6}[kind]
    c["parts"] = _log(rng, 1, max(1, min(1024, int(most // per))))
    if kind == "plan":
        c["bins"] = _log(rng, 1000, 32768)
    if kind == "eval":
        c["checked"] = rng.random() < 0.7
    if kind == "mbo":
        batch = rng.randint(4, 48)
        c.update(obs=rng.randint(8, 256), members=rng.randint(3, 8), batch=batch)
    return c


def _grid(n):
    return tuple(float(x) for x in np.linspace(1005.0, 1980.0, n)) if n > 1 else (1980.0,)


def _space(c):
    """The candidate axes of a case: SM choices spread over 1 .. 32 of the modelled GPU."""
    S = c["sms"]
    sms = tuple(int(x) for x in np.unique(np.linspace(32 / S, 32, S).round().astype(int)))
    return I.Space(c.get("parts", c.get("types", 1)), c["kernels"], c.get("comm", 1), c["pos"],
                   sms, _grid(c["freqs"]))


def _tables(c, seed):
    sp = _space(c)
    tab = I.make_tables(sp, seed=1000 + seed, comm_bytes=(4e6, 128e6))
    return sp, [torch.from_numpy(tab[k]).cuda() for k in ("t", "pw", "tc", "pc")]


def _segments(sp):
    return np.arange(sp.n_parts * sp.n_freq + 1, dtype=np.int64) * sp.cand_per_freq


def _frontier_points(c, seed):
    off, T, E = I.compose_frontiers(seed=1000 + seed, n_parts=c["parts"], n_min=c["lo"],
                                    n_max=c["hi"])
    return [torch.from_numpy(x).cuda() for x in (off, T, E)]


def _composed(P, B, n):
    """Kept buffers of a composition (entries that a call does not write stay zero)."""
    z = lambda dt, *s: torch.zeros(s, dtype=dt, device="cuda")  # noqa: E731
    f, i = torch.float64, torch.int32
    return kr.Composed(z(f, B), z(i, P, B), z(i, P, B), z(i, n), z(f, 2), z(i, 1), z(i, B),
                       z(f, B), z(f, B), z(i, 1), z(i, 1))


def _room(parts):
    """Frontier points of all partitions together that the planner's arrays hold."""
    return 4096 + 1024 * parts


def _arrays(n):
    return [torch.zeros(n, dtype=t, device="cuda")
            for t in (torch.int32, torch.float64, torch.float64)]


def _keep(arrays, fr):
    for a, x in zip(arrays, (fr.idx, fr.T, fr.E)):
        a[:x.numel()].copy_(x)
    return dict(off=fr.off, idx=arrays[0], T=arrays[1], E=arrays[2])


def _microbatch(c, seed):
    sp, d = _tables(c, seed)
    T, E = kr.evaluate_partition(sp, *d)
    fr = kr.pareto_filter(T.reshape(-1), E.reshape(-1), _segments(sp))
    cT, cE = I.microbatch_components(2000 + seed, c["comps"], sp.freqs_mhz)
    comp = [torch.from_numpy(cT).cuda(), torch.from_numpy(cE).cuda()] if c["comps"] else [None] * 2
    seg, K, F = fr.off.cpu().numpy(), sp.n_parts, sp.n_freq
    out = kr.microbatch_buffers(seg, K, F * c["bins"] if c["kind"] == "grid" else ENUM_CAP)
    for x in (out.T, out.E, out.f, out.choice):
        x.zero_()
    return dict(seg=seg, T=fr.T.clone(), E=fr.E.clone(), K=K, F=F,
                seq=list(range(K)) * c["layers"], comp=comp, out=out)


def _timing_ops(c, seed):
    block = [0] * c["before"] + [1] + [0] * c["after"] + [1]
    sp = I.Space(c["parts"], 2 * (c["before"] + c["after"]), 2, 2,
                 tuple(int(x) for x in np.linspace(4, 32, c["sms"]).round()), _grid(c["freqs"]))
    tab = I.make_tables(sp, seed=1000 + seed, comm_bytes=(8e6, 512e6))
    k1, k2, ops, _ = I.dp_instances(I.Workload(space=sp, **tab), range(sp.n_parts), block)
    return k1, k2, torch.from_numpy(ops).cuda()


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("plan", "eval", "points"):
        s["space"], s["tables"] = _tables(case, seed)
        if kind == "points":
            s["seg"] = _segments(s["space"])
            s["kept"] = _arrays(_room(case["parts"]))
        elif kind == "eval":
            s["kept"] = _arrays(_room(case["parts"]))
        else:
            s["out"] = _composed(case["parts"], case["bins"], _room(case["parts"]))
    elif kind == "compose":
        s["off"], s["T"], s["E"] = _frontier_points(case, seed)
        s["out"] = _composed(case["parts"], case["bins"], case["parts"] * case["hi"])
    elif kind == "mbo":
        sp, d = _tables(case, seed)
        T, E = kr.evaluate_partition(sp, *d)
        s["T"], s["E"] = T.reshape(-1), E.reshape(-1)
        n, P = s["T"].numel(), sp.n_parts
        oo, idx, z = I.mbo_observations(3000 + seed, [sp.n_cand] * P, case["obs"])
        s["obs_off"], s["obs_idx"] = torch.from_numpy(oo).cuda(), torch.from_numpy(idx).cuda()
        s["cand_off"] = torch.arange(P + 1, dtype=torch.int64, device="cuda") * sp.n_cand
        g = s["obs_idx"] + torch.arange(P, device="cuda").repeat_interleave(case["obs"]) * sp.n_cand
        z = torch.from_numpy(z).cuda()
        s["To"] = I.perturb(s["T"][g], z[:, 0].contiguous(), 0.02)
        s["Eo"] = I.perturb(s["E"][g], z[:, 1].contiguous(), 0.02)
        gen = torch.Generator("cuda").manual_seed(4000 + seed)
        for k, v in (("Tm", s["T"]), ("Em", s["E"])):
            u = torch.rand((case["members"], n), dtype=torch.float64, device="cuda", generator=gen)
            s[k] = u.mul_(0.1).add_(0.95).mul_(v)
        s["out"] = kr.HviScores(torch.zeros((3, n), dtype=torch.float64, device="cuda"),
                                torch.zeros((P, 3), dtype=torch.float64, device="cuda"),
                                torch.zeros((P, 4), dtype=torch.float64, device="cuda"),
                                torch.zeros(1, dtype=torch.int32, device="cuda"))
        s["unc"] = torch.zeros(n, dtype=torch.float64, device="cuda")
        b = case["batch"]
        s["k"] = [int(round(0.4 * b)), int(round(0.2 * b)), int(round(0.2 * b)), b]
        s["sel"] = kr.Batch(torch.full((P, b), -1, dtype=torch.int64, device="cuda"),
                            torch.zeros(P, dtype=torch.int32, device="cuda"),
                            torch.zeros(1, dtype=torch.int32, device="cuda"))
    elif kind in ("grid", "enum"):
        s.update(_microbatch(case, seed))
    elif kind == "timing":
        s["k1"], s["k2"], s["ops"] = _timing_ops(case, seed)
        n, ops = s["ops"].shape[0], len(s["k1"]) + len(s["k2"])
        f = dict(dtype=torch.float64, device="cuda")
        i = dict(dtype=torch.int32, device="cuda")
        s["out"] = kr.LaunchFrontier(torch.zeros((n, 64), **f), torch.zeros((n, 64), **f),
                                     torch.zeros((n, 64, ops), **i) if case["sched"] else None,
                                     torch.zeros(n, **i), torch.zeros(1, **i))
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "eval":
        fr = kr.evaluate_and_filter(s["space"], *s["tables"],
                                    validate=None if c["checked"] else False)
        return _keep(s["kept"], fr)
    if kind == "points":
        T, E = kr.evaluate_partition(s["space"], *s["tables"])
        return dict(Tall=T, Eall=E, **_keep(s["kept"], kr.pareto_filter(T, E, s["seg"])))
    if kind in ("plan", "compose"):
        if kind == "plan":
            fr = kr.evaluate_and_filter(s["space"], *s["tables"])
            pts, n_q = (fr.off, fr.T, fr.E), QUERIES
        else:
            fr, pts, n_q = None, (s["off"], s["T"], s["E"]), 1
        comp = kr.compose_frontiers(*pts, c["bins"], out=s["out"])
        ch, cand, Ts, Es, ok = kr.extract_schedule(comp, *pts, comp.stair_bin[:n_q],
                                                   cand_idx=fr.idx if fr else None)
        return dict(off=pts[0], F=comp.F, bp=comp.bp, bp_off=comp.bp_off, bin=comp.pt_bin,
                    info=comp.info, L=comp.L, n=comp.n_stair, status=comp.status,
                    stair=[comp.stair_bin, comp.stair_Tlo, comp.stair_E], choice=ch, cand=cand,
                    Tsum=Ts, Esum=Es, ok=ok)
    if kind == "mbo":
        sc = kr.hvi_scores(s["cand_off"], s["T"], s["E"], s["obs_off"], s["To"], s["Eo"], P_STATIC,
                           out=s["out"])
        u = kr.uncertainty(s["Tm"], s["Em"], out=s["unc"])
        b = kr.select_batch(s["cand_off"], sc.hvi, u, s["obs_off"], s["obs_idx"], *s["k"],
                            out=s["sel"])
        return dict(hvi=sc.hvi, hv=sc.hv, ref=sc.ref, unc=u, sel=b.sel, count=b.count)
    if kind in ("grid", "enum"):
        args = (s["seg"], s["T"], s["E"], s["K"], s["F"], s["seq"], *s["comp"])
        if kind == "grid":
            kr.microbatch_frontier(*args, n_bins=c["bins"], out=s["out"])
        else:
            kr.microbatch_enumerate(*args, cap=ENUM_CAP, out=s["out"])
        o = s["out"]
        return dict(T=o.T, E=o.E, f=o.f, choice=o.choice, n=o.n)
    r = kr.launch_timing_frontier(s["k1"], s["k2"], s["ops"], P_STATIC, c["kmax"],
                                  sched=c["sched"], out=s["out"])
    return dict(T=r.T, E=r.E, n=r.n, **({"sched": r.sched} if c["sched"] else {}))


def work(case):
    """Inputs read once, outputs written once; the arithmetic a pass cannot leave out."""
    c, kind = case, case["kind"]
    if kind in ("plan", "eval", "points"):
        sp = _space(c)
        S, slabs = sp.n_sm, sp.n_parts * sp.n_freq
        tab = 16 * slabs * (c["kernels"] * (S + 1) + c["comm"] * S)
        n = sp.n_parts * sp.n_cand
        w = dict(bytes=tab, flops=(20 if c["comm"] == 1 else 14) * n)
        if kind == "points":
            w["bytes"] += 16 * n
        if kind == "plan":
            w["bytes"] += 8 * c["parts"] * c["bins"]
            w["flops"] += 2 * c["bins"] * c["parts"] * 10
        return w
    if kind == "compose":
        n = (c["lo"] + c["hi"]) / 2
        pairs = c["parts"] * c["bins"] / 2 * min(n, c["bins"] / c["parts"] + 1)
        return dict(bytes=16 * n * c["parts"] + 8 * c["parts"] * c["bins"], flops=2 * pairs)
    if kind == "mbo":
        n = c["parts"] * _space(c).n_cand
        return dict(bytes=(16 + 16 * c["members"] + 32) * n, flops=(30 + 8 * c["members"]) * n)
    if kind in ("grid", "enum"):
        F, K = c["freqs"], c["types"]
        steps = F * (c["bins"] if kind == "grid" else 1) * K
        return dict(bytes=16 * F * K * 4 + 16 * F * c["comps"] + 24 * F * 8,
                    flops=2 * steps * 3 + F * 8 * 2 * K * c["layers"])
    ops = 2 * (c["before"] + c["after"] + 2)
    n = c["parts"] * c["freqs"] * c["sms"]
    cells = (ops // 2 + 1) ** 2 - 1
    return dict(bytes=n * (32 * ops + 4 + 2 * (16 + (4 * ops if c["sched"] else 0))),
                flops=n * cells * 60)


def tolerance(case):
    """The library fixes the order of every fp64 operation (its results are reproducible bit
    for bit), except for the scores of the optimisation: the area that a candidate adds and
    its members' deviations may be summed in another order.  Against the plain 64-bit forms
    below the scores come out equal and the uncertainty is off by 1e-15 (2-norm)."""
    if case["kind"] == "mbo":
        return {"rel": 4e-15, "max": 1e-13, "differ": 1e-4}
    return "exact"


# ---- the same results in plain torch / numpy (64 bits) ----------------------------------


def _walk(t, pw, tc, pc, pos, sm):
    """Time and energy [Q][C] of candidates (launch positions pos[m], SM choices sm[m], each
    [C]) over slabs t, pw [Q][N][S+1] and tc, pc [Q][M][S]."""
    Q, N, S1 = t.shape
    C = pos[0].numel()
    dev = t.device
    zero = torch.zeros((Q, 1, S1), dtype=t.dtype, device=dev)
    A = torch.cat([zero, t.cumsum(1)], 1).reshape(Q, -1)
    B = torch.cat([zero, (pw * t).cumsum(1)], 1).reshape(Q, -1)
    t, pw = (torch.cat([x, x[:, -1:]], 1).reshape(Q, -1) for x in (t, pw))  # row N: unused
    at = lambda x, i, s: x.gather(1, i * S1 + s)  # noqa: E731
    i = torch.zeros((Q, C), dtype=torch.int64, device=dev)
    w = torch.ones((Q, C), dtype=t.dtype, device=dev)
    Ec, tau = torch.zeros_like(w), torch.zeros_like(w)
    live = torch.ones_like(w, dtype=torch.bool)
    T = torch.zeros_like(w)

    def advance(s, budget, stop, on):
        """Compute in state s for `budget` seconds or up to kernel `stop`, where `on`."""
        nonlocal i, w, Ec
        part = on & (w < 1.0)
        need = w * at(t, i, s)
        cut = part & (need > budget)  # the kernel in progress outlasts the budget
        Ec = torch.where(part, Ec + at(pw, i, s) * torch.minimum(need, budget), Ec)
        w = torch.where(cut, (w - budget / at(t, i, s)).clamp_min(0.0), torch.where(part, 1.0, w))
        used = torch.where(part & ~cut, need, 0.0)
        i = torch.where(part & ~cut, i + 1, i)
        go = on & ~cut
        rb = budget - used
        lo, hi, base = i, torch.maximum(i, stop), at(A, i, s)
        for _ in range(N.bit_length() + 1):
            mid = (lo + hi + 1) // 2
            ok = at(A, mid, s) - base <= rb
            lo, hi = torch.where(ok, mid, lo), torch.where(ok, hi, mid - 1)
            hi = torch.maximum(lo, hi)
        done = go & (lo == stop)
        Ec = torch.where(go, Ec + (at(B, lo, s) - at(B, i, s)), Ec)
        r = rb - (at(A, lo, s) - base)
        mid = go & ~done
        Ec = torch.where(mid, Ec + at(pw, lo, s) * r, Ec)
        w = torch.where(mid, (1.0 - r / at(t, lo, s)).clamp_min(0.0), w)
        el = torch.where(done, used + (at(A, lo, s) - base), budget)
        i = torch.where(go, lo, i)
        return done, el

    s0 = torch.zeros((Q, C), dtype=torch.int64, device=dev)
    inf = torch.full_like(w, 1e300)
    end = torch.full_like(i, N)
    cm = [(tc[:, m][:, sm[m]], pc[:, m][:, sm[m]]) for m in range(len(pos))]
    for m in range(len(pos)):
        p = pos[m].expand(Q, C)
        on = live & (i < p)
        _, el = advance(s0, inf, p, on)
        tau = torch.where(on, tau + el, tau)
        fin, _ = advance((sm[m] + 1).expand(Q, C), cm[m][0], end, live)
        fin = fin & live
        tau = tau + cm[m][0]
        rest = tau
        for q in range(m + 1, len(pos)):
            rest = rest + cm[q][0]
        T = torch.where(fin, rest, T)
        live = live & ~fin
    _, el = advance(s0, inf, end, live)
    T = torch.where(live, tau + el, T)
    E = P_STATIC * T + Ec
    for a, b in cm:
        E = E + b * a
    return T, E


def _candidates(sp, device):
    """Launch positions and SM choices of one frequency's candidates, in index order."""
    if sp.n_comm == 1:
        ax = [(p, s) for p in range(sp.n_pos) for s in range(sp.n_sm)]
        x = torch.tensor(ax, device=device)
        return [x[:, 0]], [x[:, 1]]
    pairs = [(p, q) for p in range(sp.n_pos) for q in range(p, sp.n_pos)]
    x = torch.tensor(pairs, device=device).repeat_interleave(sp.n_sm ** 2, 0)
    s = torch.arange(sp.n_sm ** 2, device=device).repeat(len(pairs))
    return [x[:, 0], x[:, 1]], [s // sp.n_sm, s % sp.n_sm]


def _evaluate(sp, tables):
    """T, E [C] of every candidate, partition by partition."""
    pos, sm = _candidates(sp, tables[0].device)
    step = max(1, 3_000_000 // pos[0].numel())
    for p in range(sp.n_parts):
        got = [_walk(*(x[p, f:f + step] for x in tables), pos, sm)
               for f in range(0, sp.n_freq, step)]
        yield torch.cat([g[0].reshape(-1) for g in got]), torch.cat([g[1].reshape(-1) for g in got])


def _front(T, E):
    """Indices of the frontier of a point set, in ascending time."""
    o = torch.sort(E, stable=True).indices
    o = o[torch.sort(T[o], stable=True).indices]
    e = E[o]
    best = torch.cat([e.new_full((1,), math.inf), torch.cummin(e, 0).values[:-1]])
    return o[e < best]


def _frontiers(points):
    off, T, E = [0], [], []
    for t, e in points:
        k = _front(t, e)
        off.append(off[-1] + k.numel())
        T.append(t[k])
        E.append(e[k])
    return off, torch.cat(T), torch.cat(E)


def _padded(x, n):
    return torch.cat([x, x.new_zeros(n - x.numel())])


def _compose(off, T, E, B, used=None):
    """Bins of every point, F and back-pointers of the composition (torch, any device)."""
    P = len(off) - 1
    Tk = [T[off[k]:off[k + 1]] for k in range(P)]
    tmin, tmax = [float(x.min()) for x in Tk], [float(x.max()) for x in Tk]
    total = 0.0
    for a, b in zip(tmin, tmax):
        total += b - a
    delta = total / (B - 1) if total > 0 else 1.0
    while 1 + sum(math.floor((b - a) / delta) for a, b in zip(tmin, tmax)) > B:
        delta = math.nextafter(delta, math.inf) if hasattr(math, "nextafter") else \
            float(np.nextafter(delta, np.inf))
    F = T.new_full((B,), math.inf)
    bins, bps = [], []
    for k in range(P):
        b = torch.floor((Tk[k] - tmin[k]) / delta).to(torch.int64)
        bins.append(b)
        least = {}
        for j, (bj, ej) in enumerate(zip(b.tolist(), E[off[k]:off[k + 1]].tolist())):
            if bj not in least or ej < least[bj][0]:
                least[bj] = (ej, j)
        new, bp = torch.full_like(F, math.inf), torch.full((B,), -1, device=T.device)
        if k == 0:
            for bj, (ej, j) in least.items():
                new[bj], bp[bj] = ej, j
        else:
            for bj, (ej, j) in sorted(least.items()):
                x = F[:B - bj] + ej
                if used is None:
                    torch.minimum(new[bj:], x, out=new[bj:])
                else:
                    better = x < new[bj:]
                    bp[bj:][better] = j
                    new[bj:] = torch.where(better, x, new[bj:])
        F = new
        bps.append(bp)
    return F, bins, bps


def _exact_microbatch(case, seed):
    sp, d = _tables(case, seed)
    K, Fq = sp.n_parts, sp.n_freq
    cT, cE = I.microbatch_components(2000 + seed, case["comps"], sp.freqs_mhz)
    front = {}
    for t, (T, E) in enumerate(_evaluate(sp, d)):
        for f in range(Fq):
            s = slice(f * sp.cand_per_freq, (f + 1) * sp.cand_per_freq)
            k = _front(T[s], E[s])
            front[t, f] = (T[s][k].cpu(), E[s][k].cpu())
    if case["kind"] == "enum" and sum(
            math.prod(len(front[t, f][0]) for t in range(K)) for f in range(Fq)) > 200_000:
        return None
    outT, outE = [], []
    for f in range(Fq):
        pts = [front[t, f] for t in range(K)]
        if case["kind"] == "enum":
            picks = itertools.product(*(range(len(p[0])) for p in pts))
        else:
            n = float(case["layers"])
            off = np.concatenate([[0], np.cumsum([len(p[0]) for p in pts])])
            F, bins, bps = _compose(off, torch.cat([p[0] for p in pts]) * n,
                                    torch.cat([p[1] for p in pts]) * n, case["bins"], used=True)
            best = torch.cat([F.new_full((1,), math.inf), torch.cummin(F, 0).values[:-1]])
            picks = []
            for b in torch.nonzero(F < best).reshape(-1).tolist():
                pick = [0] * K
                for t in range(K - 1, -1, -1):
                    pick[t] = int(bps[t][b])
                    b -= int(bins[t][pick[t]])
                picks.append(pick)
        for pick in picks:
            for out, x, comp in ((outT, 0, cT), (outE, 1, cE)):
                v = [float(pts[t][x][pick[t]]) for t in range(K)] * case["layers"]
                out.append(math.fsum(v + [float(comp[i, f]) for i in range(case["comps"])]))
    T, E = torch.tensor(outT, dtype=torch.float64), torch.tensor(outE, dtype=torch.float64)
    k = _front(T, E)
    n = Fq * case["bins"] if case["kind"] == "grid" else ENUM_CAP
    return dict(T=_padded(T[k], n), E=_padded(E[k], n), f=None, choice=None, n=None)


def _exact_mbo(case, seed):
    s = prepare(case, seed)
    P, n = case["parts"], s["T"].numel() // case["parts"]
    hvi = torch.zeros((3, P * n), dtype=torch.float64, device="cuda")
    hv, ref = [], []
    for p in range(P):
        o = slice(p * case["obs"], (p + 1) * case["obs"])
        To, Eo = s["To"][o], s["Eo"][o]
        T, E = s["T"][p * n:(p + 1) * n], s["E"][p * n:(p + 1) * n]
        rT = 1.1 * float(To.max())
        row, h = [rT], []
        for v in range(3):
            eo, e = ((Eo, E), (Eo - P_STATIC * To, E - P_STATIC * T),
                     (P_STATIC * To, P_STATIC * T))[v]
            rE = 1.1 * float(eo.max())
            k = _front(To, eo)
            ts, es = [-math.inf] + To[k].tolist() + [rT], [rE] + eo[k].tolist()
            h.append(sum((ts[i + 1] - ts[i]) * (rE - es[i]) for i in range(1, len(es))))
            acc = torch.zeros_like(T)
            for i in range(len(es)):
                wide = (min(ts[i + 1], rT) - T.clamp_min(ts[i])).clamp_min(0.0)
                acc += wide * (es[i] - e).clamp_min(0.0)
            hvi[v, p * n:(p + 1) * n] = acc
            row.append(rE)
        hv.append(h)
        ref.append(row)
    unc = s["Tm"].std(0, correction=0) + s["Em"].std(0, correction=0)
    return dict(hvi=hvi, hv=torch.tensor(hv, dtype=torch.float64),
                ref=torch.tensor(ref, dtype=torch.float64), unc=unc, sel=None, count=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "timing":
        return None  # a dynamic program over point sets: minutes in plain Python
    if kind == "mbo":
        return _exact_mbo(case, seed)
    if kind in ("grid", "enum"):
        return _exact_microbatch(case, seed)
    if kind == "compose":
        off, T, E = _frontier_points(case, seed)
        F, _, _ = _compose(off.tolist(), T, E, case["bins"])
        return dict(F=F)
    sp, d = _tables(case, seed)
    if kind == "points":
        Cf = sp.cand_per_freq
        both = list(_evaluate(sp, d))
        off, T, E = _frontiers((t[x:x + Cf], e[x:x + Cf]) for t, e in both
                               for x in range(0, sp.n_cand, Cf))
        n = _room(case["parts"])
        return dict(Tall=torch.stack([x[0] for x in both]), Eall=torch.stack([x[1] for x in both]),
                    T=_padded(T, n), E=_padded(E, n))
    off, T, E = _frontiers(_evaluate(sp, d))
    if kind == "eval":
        n = _room(case["parts"])
        return dict(T=_padded(T, n), E=_padded(E, n))
    F, _, _ = _compose(off, T.cpu(), E.cpu(), case["bins"])
    return dict(F=F)
