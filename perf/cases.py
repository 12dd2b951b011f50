"""The measured workloads of this framework: the calls that a user of libargus makes, over the sizes they make them at.

A monitoring job holds one window of kernel events in HBM and calls summarize on it; cross-rank, iteration windows and
the group comparison then run over the summaries, the KDE and W1 steps over the events and their clusters, and the
record stream is what leaves the GPU. Shapes follow the five workloads of the benchmark (tiny, medium, production,
cluster, skew); the cluster step's events are cut to 2,048 of its 10,240 ranks (1,024 for the KDE), so that a window
and its workspace fit the card three times over, while the per-cell steps (cross-rank, W1, L2, records) keep all
10,240 ranks. Inputs are made on the GPU from the seed alone: one template of kernel launches per job, repeated in
every rank-step, with lognormal durations, Zipf-distributed ids, multimodal kernels, stragglers and degraded pairs.
"""
import math

import numpy as np
import torch

import paper_2606_20374_amd as pa

DEV = "cuda"
NB = 32                              # octave bins of a summary cell
EPOCH_NS = 1_764_000_000_000_000_000
I64_MAX, I64_MIN = 2**63 - 1, -(2**63)


def listed():
    return [
        # the smallest use: eight ranks' window through every step, where launches and latency are all there is
        {"name": "pipeline_tiny", "path": "pipeline", "ranks": 8, "steps": 4, "events": 20_000, "kernels": 64,
         "streams": 4, "ids": "uniform", "ragged": False, "invalid_ppm": 0},
        # an ordinary window of a mid-sized job: rank-steps of uneven length with some corrupted records
        {"name": "summarize_medium_ragged", "path": "summarize", "ranks": 256, "steps": 8, "events": 100_000,
         "kernels": 512, "streams": 8, "ids": "zipf", "ragged": True, "invalid_ppm": 200},
        # the whole-cluster step's rank-steps: the stream that the whole path is paced by
        {"name": "summarize_cluster", "path": "summarize", "ranks": 2048, "steps": 1, "events": 400_000,
         "kernels": 2048, "streams": 16, "ids": "zipf", "ragged": False, "invalid_ppm": 0},
        # a sparse id space whose events go to a few hot communication kernels (mapped slots)
        {"name": "summarize_skew", "path": "summarize", "ranks": 1024, "steps": 4, "events": 200_000,
         "kernels": 8200, "streams": 16, "ids": "skew", "ragged": False, "invalid_ppm": 0},
        # the paper's own grouping key, (kernel, stream), on production rank-steps: 32,768 keys
        {"name": "summarize_keyed", "path": "keyed", "ranks": 512, "steps": 1, "events": 400_000, "kernels": 2048,
         "streams": 16, "ids": "zipf", "ragged": False, "invalid_ppm": 0},
        # straggler detection over the whole cluster's summaries
        {"name": "cross_rank_cluster", "path": "cross_rank", "ranks": 10_240, "steps": 1, "kernels": 2048},
        # step-time windows over a long run
        {"name": "l1_long", "path": "iter_windows", "ranks": 10_240, "steps": 1000},
        # duration clusters of a production step
        {"name": "kde_production", "path": "kde", "ranks": 1024, "steps": 1, "events": 400_000, "kernels": 2048,
         "streams": 16, "ids": "zipf", "ragged": False, "invalid_ppm": 0},
        # duration clusters of a sparse id space with long-tailed hot kernels, ragged, some records corrupted
        {"name": "kde_skew_ragged", "path": "kde", "ranks": 256, "steps": 4, "events": 200_000, "kernels": 8200,
         "streams": 16, "ids": "skew", "ragged": True, "invalid_ppm": 200},
        # cross-rank deviation of the whole cluster's duration clusters
        {"name": "w1_cluster", "path": "w1", "ranks": 10_240, "steps": 1, "kernels": 2048, "grid": 64},
        # group-aware comparison of the whole cluster (tensor 8, pipeline 8, expert 8)
        {"name": "l2_cluster", "path": "l2", "ranks": 10_240, "steps": 1, "kernels": 2048, "tp": 8, "pp": 8, "ep": 8},
        # the record stream of the whole cluster's summaries
        {"name": "compact_cluster", "path": "compact", "ranks": 10_240, "steps": 1, "kernels": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["pipeline", "summarize", "summarize", "keyed", "cross_rank", "iter_windows", "kde", "kde", "w1",
                       "l2", "compact"])
    if path == "pipeline":
        return {"path": path, "ranks": _log_int(rng, 4, 64), "steps": _log_int(rng, 1, 8),
                "events": _log_int(rng, 2_000, 40_000), "kernels": _log_int(rng, 20, 500), "streams": rng.randint(1, 16),
                "ids": rng.choice(["uniform", "zipf"]), "ragged": rng.random() < 0.5,
                "invalid_ppm": rng.choice([0, 200])}
    if path in ("summarize", "keyed", "kde"):
        ids = rng.choice(["uniform", "zipf", "zipf", "skew"])
        kernels = _log_int(rng, 2_100, 9_000) if ids == "skew" else _log_int(rng, 64, 2_048)
        streams = rng.randint(1, 16)
        if path == "keyed":
            streams = max(1, min(streams, 60_000 // kernels))
        events = _log_int(rng, 5_000, 400_000)
        total = _log_int(rng, 2_000_000, 400_000_000 if path == "summarize" else 200_000_000)
        segs = max(1, min(total // events, 150_000_000 // kernels))
        steps = rng.choice([1, 1, 2, 5, 8])
        return {"path": path, "ranks": max(1, segs // steps), "steps": steps, "events": events, "kernels": kernels,
                "streams": streams, "ids": ids, "ragged": rng.random() < 0.5, "invalid_ppm": rng.choice([0, 0, 200])}
    if path == "iter_windows":
        steps = _log_int(rng, 8, 4_000)
        return {"path": path, "ranks": _log_int(rng, 8, min(10_240, 10_240_000 // steps)), "steps": steps}
    ranks, steps = _log_int(rng, 8, 10_240), rng.choice([1, 1, 2, 4])
    kernels = _log_int(rng, 50, max(60, min(4_000, 20_000_000 // (ranks * steps))))
    case = {"path": path, "ranks": ranks, "steps": steps, "kernels": kernels}
    if path == "w1":
        case["grid"] = rng.choice([32, 64, 64, 128 if ranks * steps * kernels < 8_000_000 else 64])
    if path == "l2":
        case["tp"], case["pp"], case["ep"] = rng.choice([(2, 2, 2), (2, 4, 4), (8, 4, 8), (8, 8, 8), (4, 1, 16)])
    return case


# ------------------------------------------------------------------ inputs
def _shares(ids, kernels):
    """Probability of each kernel id in the job's launch template."""
    if ids == "zipf":
        w = np.arange(1, kernels + 1, dtype=np.float64) ** -1.1
    elif ids == "skew":  # eight hot ids take nine launches in ten
        w = np.full(kernels, 0.1 / (kernels - 8))
        w[:8] = 0.9 / 8
    else:
        w = np.ones(kernels)
    return w / w.sum()


def _kernel_tables(rng, kernels):
    """Base duration of each kernel (2 us to 5 ms) and how many scales (x1, x3, x9) its launches run at."""
    base = np.exp(rng.uniform(math.log(2e3), math.log(5e6), kernels))
    modes = np.where(rng.random(kernels) < 0.3, rng.integers(2, 4, kernels), 1)
    return base, modes


def _rank_scale(g, ranks):
    """Slowdown of each rank: about one in a thousand (at least one) is a straggler."""
    scale = torch.ones(ranks, device=DEV, dtype=torch.float64)
    slow = torch.randint(ranks, (max(1, ranks // 1000),), generator=g, device=DEV)
    scale[slow] = 1.05 + 0.45 * torch.rand(len(slow), generator=g, device=DEV, dtype=torch.float64)
    return scale


def _events(case, seed):
    """One window of kernel events, as structure-of-arrays tensors on the GPU."""
    R, S, K, NS, ids = case["ranks"], case["steps"], case["kernels"], case["streams"], case["ids"]
    rng = np.random.default_rng([seed, 11])
    g = torch.Generator(device=DEV).manual_seed(seed * 8 + 1)
    G = R * S
    T = max(64, case["events"] // 10)  # launches of the template: ten training micro-steps to a window
    lens = np.full(G, case["events"], dtype=np.int64)
    if case["ragged"]:
        lens = (lens * rng.uniform(0.4, 1.6, G)).astype(np.int64)
        lens[rng.random(G) < 0.01] = 0  # a rank that reported nothing
    off = np.zeros(G + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    base, modes = _kernel_tables(rng, K)
    kid = rng.choice(K, size=T, p=_shares(ids, K))
    nominal = base[kid] * 3.0 ** np.floor(rng.random(T) * modes[kid])
    hot = (kid < 8) & (ids == "skew")
    nominal[hot] = 3e4
    at = np.zeros(T)  # launch time in the template: each stream runs back to back with 1-20 us gaps
    gaps = rng.uniform(1e3, 2e4, T)
    for st in range(NS):
        mine = kid % NS == st
        at[mine] = np.cumsum(gaps[mine] + nominal[mine]) - nominal[mine]
    span = int(at.max() + nominal.max() + 2e4)
    up = lambda x, dt: torch.from_numpy(np.ascontiguousarray(x)).to(DEV, dt)  # noqa: E731
    kid_t, nom_t, at_t, hot_t = up(kid, torch.int32), up(nominal, torch.float64), up(at, torch.int64), up(hot, torch.bool)
    scale, off_t = _rank_scale(g, R), up(off, torch.int64)
    n = int(off[-1])
    ev = {"kernel_id": torch.empty(n, dtype=torch.int32, device=DEV), "stream": torch.empty(n, dtype=torch.int32, device=DEV),
          "start_ns": torch.empty(n, dtype=torch.int64, device=DEV), "end_ns": torch.empty(n, dtype=torch.int64, device=DEV),
          "seg_off": off_t}
    g0 = 0
    while g0 < G:  # whole segments, about 32 million events at a time
        g1 = max(g0 + 1, int(np.searchsorted(off, off[g0] + 32_000_000, side="right")) - 1)
        g1 = min(G, g1)
        a, b = int(off[g0]), int(off[g1])
        if b > a:
            seg = torch.repeat_interleave(torch.arange(g0, g1, device=DEV), off_t[g0 + 1:g1 + 1] - off_t[g0:g1], output_size=b - a)
            i = torch.arange(a, b, device=DEV) - off_t[seg]
            rep, p = i // T, i % T
            swap = torch.rand(b - a, generator=g, device=DEV) < 0.05  # launches that a rank's stream reordered
            p = torch.where(swap, (p ^ 1).clamp_(max=T - 1), p)
            d = nom_t[p] * scale[seg // S] * torch.exp(0.1 * torch.randn(b - a, generator=g, device=DEV)).double()
            if ids == "skew":  # communication kernels wait for their peers: Pareto tails
                u = torch.rand(b - a, generator=g, device=DEV).clamp_(min=1e-5)
                d = torch.where(hot_t[p], 1.5e4 * u.pow(-1 / 1.5).double(), d)
            k = kid_t[p]
            start = EPOCH_NS + (seg % S) * (span * 50) + rep * span + at_t[p]
            end = start + d.to(torch.int64)
            stream = k % NS
            if case["invalid_ppm"]:
                bad = torch.rand(b - a, generator=g, device=DEV) * 1e6 < case["invalid_ppm"]
                which = torch.randint(3, (b - a,), generator=g, device=DEV)
                k = torch.where(bad & (which == 0), -1, k)
                end = torch.where(bad & (which == 1), start - 1, end)
                stream = torch.where(bad & (which == 2), NS, stream)
            ev["kernel_id"][a:b], ev["stream"][a:b], ev["start_ns"][a:b], ev["end_ns"][a:b] = k, stream, start, end
        g0 = g1
    return ev


def _summary_buffers(R, S, cells, NS):
    """Output buffers of summarize, filled with the identity values that absent cells keep."""
    s = pa.alloc_summary(R, S, cells, NS, DEV)
    for f, v in (("sum_ns", 0), ("min_ns", I64_MAX), ("max_ns", I64_MIN), ("hist", 0)):
        s[f].fill_(v)
    return s


def _cells(case, seed):
    """Launch counts [K] (one template: the same in every rank), kernel tables and rank slowdowns of a job whose
    summaries are made directly: 400,000 events to a rank-step, some ids never launched."""
    K = case["kernels"]
    rng = np.random.default_rng([seed, 12])
    g = torch.Generator(device=DEV).manual_seed(seed * 8 + 2)
    base, modes = _kernel_tables(rng, K)
    n = rng.multinomial(40_000, _shares("zipf", K)) * 10
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
    return rng, g, up(n), up(base), up(modes), _rank_scale(g, case["ranks"])


def _summaries(case, seed, full=False):
    """count and sum_ns of every cell; with full also min_ns, max_ns and the octave histogram."""
    R, S, K = case["ranks"], case["steps"], case["kernels"]
    rng, g, n, base, modes, scale = _cells(case, seed)
    shape = (R, S, K)
    z = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).double()
    lost = torch.randint(0, 50, shape, generator=g, device=DEV) == 0  # a few launches fell into the next window
    count = (n - lost.to(torch.int64) * (n > 1)).clamp_(min=0).expand(shape).contiguous()
    level = torch.where(modes > 2, 13.0 / 3, torch.where(modes > 1, 2.0, 1.0))
    pairs = torch.rand(shape, generator=g, device=DEV) < 2.5e-6  # degraded (rank, kernel) pairs
    mean = base * level * scale.view(R, 1, 1) * (1.005 + 0.1 * z / count.clamp(min=1).double().sqrt())
    mean = torch.where(pairs, mean * 1.8, mean)
    out = {"count": count.to(torch.int32).reshape(-1), "sum_ns": (mean * count).to(torch.int64).reshape(-1)}
    if full:
        # a mode's durations (sigma 0.144 octaves) fall into the octave of its median and the next one up or down
        C = R * S * K
        hist = torch.zeros(C, NB, dtype=torch.int32, device=DEV)
        left = count.to(torch.int32).reshape(C).clone()
        cnt = left.clone()
        for m in range(3):
            lg = torch.log2(base * 3.0**m)
            has = (modes > m).expand(shape).reshape(C)
            part = torch.where(has, torch.where((modes == m + 1).expand(shape).reshape(C), left, (cnt // modes.expand(shape).reshape(C)).to(torch.int32)), 0)
            part = torch.minimum(part, left)
            left = left - part
            up_share = torch.special.ndtr((lg - torch.floor(lg) - 1) / 0.144).expand(shape).reshape(C)
            dn_share = torch.special.ndtr((torch.floor(lg) - lg) / 0.144).expand(shape).reshape(C)
            u = torch.rand(C, generator=g, device=DEV)
            hi = torch.floor(part * up_share + u).to(torch.int32)
            lo = torch.floor(part * dn_share + u).to(torch.int32)
            hi = torch.minimum(hi, part)
            lo = torch.minimum(lo, part - hi)
            bin0 = torch.floor(lg).to(torch.int64).expand(shape).reshape(C, 1)
            for b, v in ((0, part - hi - lo), (1, hi), (-1, lo)):
                hist.scatter_add_(1, bin0 + b, v.view(C, 1))
        gone = out["count"] == 0
        low, top = mean.reshape(-1) / level.expand(shape).reshape(-1), mean.reshape(-1) * 1.3
        out["hist"] = hist.reshape(-1)
        out["sum_ns"][gone] = 0
        out["min_ns"] = torch.where(gone, I64_MAX, (low * 0.75).to(torch.int64))
        out["max_ns"] = torch.where(gone, I64_MIN, top.to(torch.int64))
    return out


def _clusters(case, seed):
    """Duration clusters of every cell, as the KDE step reports them: one per mode of the kernel, (count, p50, p99)
    with the sampling noise of the cell's launches; a few cells merged two modes into one cluster."""
    R, S, K = case["ranks"], case["steps"], case["kernels"]
    rng, g, n, base, modes, scale = _cells(case, seed)
    shape = (R, S, K)
    C = R * S * K
    n_c, modes_c = n.expand(shape).reshape(C), modes.expand(shape).reshape(C)
    base_c = (base * scale.view(R, 1, 1)).expand(shape).reshape(C)
    found = torch.where(torch.rand(C, generator=g, device=DEV) < 0.03, (modes_c - 1).clamp(min=1), modes_c)
    found = torch.where(n_c >= 3 * found, found, torch.ones_like(found))
    found = torch.where(n_c > 0, found, torch.zeros_like(found))
    cl = {"n_clusters": found.to(torch.uint8), "count": torch.zeros(C, 4, dtype=torch.int32, device=DEV),
          "p50_ns": torch.zeros(C, 4, dtype=torch.int64, device=DEV), "p99_ns": torch.zeros(C, 4, dtype=torch.int64, device=DEV)}
    left = n_c.clone()
    for m in range(3):
        on = found > m
        cnt = torch.where(found == m + 1, left, n_c // found.clamp(min=1))
        cnt = torch.where(on, cnt, torch.zeros_like(cnt))
        left = left - cnt
        noise = 1 / cnt.clamp(min=1).double().sqrt()
        med = base_c * 3.0**m * torch.exp(0.125 * noise * torch.randn(C, generator=g, device=DEV).double())
        # the nearest-rank 99th percentile: the largest of few samples, else 2.33 sigma with its own noise
        tail = torch.minimum(torch.full_like(noise, 2.326), 1.2 * torch.log1p(cnt.double()) ** 0.75)
        tail = torch.where(cnt < 2, torch.zeros_like(tail), tail)
        p99 = med * torch.exp((0.1 * tail + 0.3 * noise * torch.randn(C, generator=g, device=DEV).double()).clamp(min=0))
        p99 = torch.where(cnt < 2, med, p99)
        cl["count"][:, m] = cnt.to(torch.int32)
        cl["p50_ns"][:, m] = torch.where(on, med, torch.zeros_like(med)).to(torch.int64)
        cl["p99_ns"][:, m] = torch.where(on, p99, torch.zeros_like(med)).to(torch.int64)
    return {f: v.reshape(-1) for f, v in cl.items()}


def _step_times(case, seed):
    """Step times of each rank: 1 s with 4% noise, a 1.5x regression from some step on in every seventh rank, a 3x
    spike in every eleventh."""
    R, S = case["ranks"], case["steps"]
    g = torch.Generator(device=DEV).manual_seed(seed * 8 + 3)
    y = 1e9 * (1 + 0.04 * torch.randn(R, S, generator=g, device=DEV, dtype=torch.float64))
    t = torch.arange(S, device=DEV)
    since = torch.randint(S // 3, S, (R, 1), generator=g, device=DEV)
    spike = torch.randint(S, (R, 1), generator=g, device=DEV)
    r = torch.arange(R, device=DEV).view(R, 1)
    y = torch.where((r % 7 == 0) & (t >= since), y * 1.5, y)
    y = torch.where((r % 11 == 0) & (t == spike), y * 3.0, y)
    return y.to(torch.int64).reshape(-1)


def _groups(ranks, kernels, tp, pp, ep, seed):
    """Routing table of the kernels and the member lists of the tensor, pipeline, data and expert groups."""
    rng = np.random.default_rng([seed, 13])
    r = np.arange(ranks)
    t, p, d = r % tp, (r // tp) % pp, r // (tp * pp)
    keys = [d * pp + p, d * tp + t, p * tp + t, ((d // ep) * pp + p) * tp + t]
    most = max(int(k.max()) for k in keys) + 1
    off, mem = np.zeros((4, most + 1), np.int32), np.zeros((4, ranks), np.int32)
    for i, key in enumerate(keys):
        mem[i] = np.argsort(key, kind="stable")
        off[i, 1:] = np.cumsum(np.bincount(key, minlength=most))
    route = rng.choice(4, size=kernels, p=[0.15, 0.10, 0.50, 0.25]).astype(np.uint8)
    return tuple(torch.from_numpy(x).to(DEV) for x in (route, off, mem))


def prepare(case, seed):
    path, R, S = case["path"], case["ranks"], case["steps"]
    st = {"case": case, "dims": (R, S)}
    if path == "iter_windows":
        st["step_ns"], st["out"] = _step_times(case, seed), pa.alloc_iter_windows(R, S, DEV)
        return st
    K = case["kernels"]
    if path in ("cross_rank", "l2"):
        st.update(_summaries(case, seed))
    if path == "cross_rank":
        st["out"] = pa.alloc_cross_rank(R, S, K, DEV)
    elif path == "l2":
        st["groups"] = _groups(R, K, case["tp"], case["pp"], case["ep"], seed)
        st["out"] = pa.alloc_l2(R, S, K, 4, st["groups"][1].shape[1] - 1, DEV)
    elif path == "compact":
        st["summary"] = _summaries(case, seed, full=True)
        # room for a record of every cell with eight octave bins (these have up to seven)
        st["out"] = torch.zeros(R * S * K * 73, dtype=torch.uint8, device=DEV)
    elif path == "w1":
        st["clusters"], st["out"] = _clusters(case, seed), pa.alloc_w1(R, S, K, case["grid"], DEV)
    else:
        NS = case["streams"]
        st["ev"] = _events(case, seed)
        st["out"] = _summary_buffers(R, S, K * (NS if path == "keyed" else 1), NS)
        n = st["ev"]["kernel_id"].numel()
        if path == "kde":
            st["summary"] = pa.summarize(st["ev"], R, S, K, NS, out=st["out"])
            st["out"] = pa.alloc_kde(n, R, S, K, DEV)
        elif path == "pipeline":
            st["groups"] = _groups(R, K, 2, 2, 2, seed)
            st["bufs"] = {"sum": st["out"], "xr": pa.alloc_cross_rank(R, S, K, DEV), "l1": pa.alloc_iter_windows(R, S, DEV)}
            st["kde"], st["w1"] = pa.alloc_kde(n, R, S, K, DEV), pa.alloc_w1(R, S, K, 64, DEV)
            st["l2"] = pa.alloc_l2(R, S, K, 4, st["groups"][1].shape[1] - 1, DEV)
            st["bytes"] = torch.zeros(R * S * K * 200 + 64, dtype=torch.uint8, device=DEV)
    return st


def _outputs(d):
    return {f: v for f, v in d.items() if isinstance(v, torch.Tensor) and not f.startswith("_")}


def run(st):
    case = st["case"]
    path, (R, S), K = case["path"], st["dims"], case.get("kernels")
    if path == "iter_windows":
        return _outputs(pa.iter_windows(st["step_ns"], R, S, out=st["out"]))
    if path == "cross_rank":
        return _outputs(pa.cross_rank(st["count"], st["sum_ns"], R, S, K, out=st["out"]))
    if path == "l2":
        return _outputs(pa.l2(st["count"], st["sum_ns"], R, S, K, *st["groups"], out=st["out"]))
    if path == "compact":
        return _outputs(pa.compact(st["summary"], R, S, K, 0, out=st["out"]))
    if path == "w1":
        return _outputs(pa.w1(st["clusters"], R, S, K, out=st["out"], grid=case["grid"]))
    NS = case["streams"]
    if path in ("summarize", "keyed"):
        return _outputs(pa.summarize(st["ev"], R, S, K, NS, out=st["out"], keyed=path == "keyed"))
    if path == "kde":
        return _outputs(pa.kde(st["ev"], st["summary"], R, S, K, NS, out=st["out"]))
    s, x, w = pa.run_step(st["ev"], R, S, K, NS, bufs=st["bufs"])
    kd = pa.kde(st["ev"], s, R, S, K, NS, out=st["kde"])
    w1 = pa.w1(kd, R, S, K, out=st["w1"])
    l2 = pa.l2(s["count"], s["sum_ns"], R, S, K, *st["groups"], out=st["l2"])
    cp = pa.compact(s, R, S, K, 0, out=st["bytes"])
    return {"sum": _outputs(s), "xr": _outputs(x), "l1": _outputs(w), "kde": _outputs(kd), "w1": _outputs(w1),
            "l2": _outputs(l2), "cp": _outputs(cp)}


# ------------------------------------------------------------- work and bounds
def _present(case):
    """Share of a summary's cells that hold events: ids that a template of 40,000 Zipf launches has."""
    K, T = case["kernels"], max(64, case.get("events", 400_000) // 10)
    p = _shares(case.get("ids", "zipf"), K)
    return float(np.mean(1 - np.exp(T * np.log1p(-p)))) if K > 1 else 1.0


def work(case):
    path, R, S = case["path"], case["ranks"], case["steps"]
    if path == "iter_windows":
        return {"bytes": 9 * R * S + 13 * R, "flops": 40 * R * S}
    K, G = case["kernels"], R * S
    C, SK = G * K, S * K
    present = _present(case) * C
    per = {
        "cross_rank": 12 * C + 9 * C + 13 * G + 52 * SK,
        "l2": 12 * C + 5 * C + 33 * SK * (R // 2),
        "compact": 4 * C + 152 * present + 46 * present + 8 * G,
        "w1": C + 9 * C + 80 * present + 52 * SK,
    }
    if "tp" in case:
        per["l2"] = 12 * C + 5 * C + 33 * SK * math.ceil(R / min(case["tp"], case["pp"], case["ep"]))
    if path in per:
        return {"bytes": per[path], "flops": (40 * case["grid"] if path == "w1" else 40) * C}
    E = G * case["events"]
    summ = 24 * E + 156 * present + (48 + 8 * case["streams"]) * G
    if path in ("summarize", "keyed"):
        return {"bytes": summ, "flops": 10 * E}
    kde = 20 * E + (4 * E if case["invalid_ppm"] else 0) + 20 * C + 85 * C
    if path == "kde":
        return {"bytes": kde, "flops": 40 * E}
    return {"bytes": summ + kde + sum(per.values()), "flops": 100 * E}


def tolerance(case):
    # whole numbers (counts, sums, order statistics, flags, records) are exact on every path
    if case["path"] in ("summarize", "keyed", "kde", "compact"):
        return "exact"
    # floats are computed in 64 bits and rounded once to 32
    if case["path"] in ("cross_rank", "l2", "iter_windows"):
        return {"rel": 1.2e-7}
    # W1 adds 64-bit products of 16-bit CDF steps; a CDF value within rounding of a step may fall to either side
    return {"rel": 1.2e-7, "differ": 1e-6}


# ------------------------------------------------------------------- 64 bits
def _exact_cross_rank(count, total, R, S, K):
    n = (count.long() & 0xFFFFFFFF).view(R, S, K)
    x = total.view(R, S, K) // n.clamp(min=1)
    z, mean = torch.zeros(R, S, K, dtype=torch.float64, device=DEV), torch.where(n > 0, total.view(R, S, K).double() / n.clamp(min=1), 0.0)
    xmean = torch.zeros(S, K, dtype=torch.float64, device=DEV)
    for s in range(S):
        for k0 in range(0, K, 256):
            v, has = x[:, s, k0:k0 + 256], n[:, s, k0:k0 + 256] > 0
            m = has.sum(0)
            big = torch.where(has, v, I64_MAX)
            mid = ((m - 1) // 2).clamp(min=0).view(1, -1)
            med = torch.gather(torch.sort(big, 0).values, 0, mid)
            dev = torch.where(has, (v - med).abs(), I64_MAX)
            mad = torch.gather(torch.sort(dev, 0).values, 0, mid).clamp(min=1)
            fine = m >= 3
            z[:, s, k0:k0 + 256] = torch.where(has & fine, (v - med).double() / (1.4826 * mad.double()), 0.0)
            xmean[s, k0:k0 + 256] = torch.where(fine, torch.where(has, v, 0).double().sum(0) / m.clamp(min=1), 0.0)
    return {"z": z.reshape(-1), "mean_ns": mean.reshape(-1), "xmean_ns": xmean.reshape(-1)}


def _exact_l2(count, total, R, S, E, route, off, mem):
    n = (count.long() & 0xFFFFFFFF).view(R, S, E)
    x, has = (total.view(R, S, E) // n.clamp(min=1)).double(), n > 0
    most = off.shape[1] - 1
    out = {f: torch.zeros(S, E, most, dtype=torch.float64, device=DEV) for f in ("mean_ns", "std_ns", "cv")}
    z = torch.zeros(R, S, E, dtype=torch.float64, device=DEV)
    for d in range(4):
        e = torch.nonzero(route == d).view(-1)
        group = torch.repeat_interleave(torch.arange(most, device=DEV), (off[d, 1:] - off[d, :-1]).long())
        of = torch.empty(R, dtype=torch.int64, device=DEV)
        of[mem[d].long()] = group
        for s in range(S):
            v, h = x[:, s][:, e], has[:, s][:, e].double()
            add = lambda q: torch.zeros(most, len(e), dtype=torch.float64, device=DEV).index_add_(0, of, q)  # noqa: E731
            m = add(h)
            mean = add(v * h) / m.clamp(min=1)
            std = (add(((v - mean[of]) * h) ** 2) / (m - 1).clamp(min=1)).sqrt()
            ok = m >= 3
            mean, std = torch.where(ok, mean, 0.0), torch.where(ok, std, 0.0)
            out["mean_ns"][s, e], out["std_ns"][s, e] = mean.T, std.T
            out["cv"][s, e] = torch.where(mean > 0, std / mean.clamp(min=1e-300), 0.0).T
            ok_r = ok[of] & (h > 0) & (std[of] > 0)
            z[:, s, :].index_copy_(1, e, torch.where(ok_r, (v - mean[of]) / std[of].clamp(min=1e-300), 0.0))
    return {**{f: v.reshape(-1) for f, v in out.items()}, "z": z.reshape(-1)}


def _exact_iter_windows(y, R, S):
    ratio = torch.zeros(R, dtype=torch.float64, device=DEV)
    if S < 4:
        return {"cp_ratio": ratio}
    t = torch.arange(2, S - 1, device=DEV)
    y = y.view(R, S).double()
    for r0 in range(0, R, 2048):
        v = y[r0:r0 + 2048]
        centre = v.mean(1, keepdim=True)
        s1, s2 = torch.cumsum(v - centre, 1), torch.cumsum((v - centre) ** 2, 1)

        def side(n, a, b):  # mean and sample relative deviation of n points of centred sums a, b
            mean = centre + a / n
            return mean, ((b - a * a / n).clamp(min=0) / (n - 1)).sqrt() / mean

        ml, rl = side(t, s1[:, t - 1], s2[:, t - 1])
        mr, rr = side(S - t, s1[:, -1:] - s1[:, t - 1], s2[:, -1:] - s2[:, t - 1])
        ok = (mr / ml >= 1.3) & (rl <= 0.1) & (rr <= 0.1)
        ratio[r0:r0 + 2048] = torch.where(ok, mr / ml, 0.0).max(1).values
    return {"cp_ratio": ratio}


def _exact_w1(cl, R, S, K, G):
    nc, cnt = cl["n_clusters"].view(R, S, K), cl["count"].view(R, S, K, 4).double()
    out = {f: torch.zeros(S, K, dtype=torch.float64, device=DEV) for f in ("q1", "q3", "fence")}
    score = torch.zeros(R, S, K, dtype=torch.float64, device=DEV)
    on = torch.arange(4, device=DEV) < nc.unsqueeze(-1)
    p50 = cl["p50_ns"].view(R, S, K, 4).clamp(min=1)
    p99 = torch.maximum(cl["p99_ns"].view(R, S, K, 4).clamp(min=1), p50)
    for s in range(S):
        for k in range(K):
            who = torch.nonzero(nc[:, s, k] > 0).view(-1)
            n = len(who)
            if n < 3:
                continue
            a, b, w, o = p50[who, s, k], p99[who, s, k], cnt[who, s, k], on[who, s, k]
            small = int(b.max()) < 2**31  # squares fit 64 bits: the bounds are whole numbers
            if small:
                lo = torch.where(o, (a * a) // b, I64_MAX).min().clamp(min=1).double()
                hi = torch.where(o, (b * b + a - 1) // a, 0).max().double()
            else:
                lo = torch.where(o, torch.floor(a.double() ** 2 / b.double()), math.inf).min().clamp(min=1.0)
                hi = torch.where(o, torch.ceil(b.double() ** 2 / a.double()), 0.0).max()
            u = torch.log(lo) + torch.arange(G, device=DEV) * ((torch.log(hi) - torch.log(lo)) / (G - 1))
            mu = torch.log(a.double())
            sg = (torch.log(b.double()) - mu) / 2.326
            wt = torch.where(o, w, 0.0)
            wt = wt / wt.sum(1, keepdim=True)
            F = torch.zeros(n, G, dtype=torch.float64, device=DEV)
            for c in range(4):
                dev = u.view(1, G) - mu[:, c:c + 1]
                ph = 0.5 * torch.special.erfc(-dev / (sg[:, c:c + 1] * math.sqrt(2)).clamp(min=1e-300))
                F += wt[:, c:c + 1] * torch.where(sg[:, c:c + 1] > 0, ph, (dev >= 0).double())
            q = torch.floor(F * 65536).clamp(max=65535)
            v, at = torch.sort(q, 0)
            before = torch.cumsum(v, 0) - v
            i = torch.arange(n, device=DEV, dtype=torch.float64).view(n, 1)
            rows = torch.empty_like(q).scatter_(0, at, v * (2 * i - n) + v.sum(0) - 2 * before)
            x = torch.exp(u)
            g = torch.arange(G, device=DEV)
            wg = (x[(g + 1).clamp(max=G - 1)] - x[(g - 1).clamp(min=0)]) / 2
            sc = (rows * wg).sum(1) / (65536.0 * (n - 1))
            score[who, s, k] = sc
            v = torch.sort(sc).values
            q1, q3 = v[(n - 1) // 4], v[3 * (n - 1) // 4]
            out["q1"][s, k], out["q3"][s, k], out["fence"][s, k] = q1, q3, q3 + 1.5 * (q3 - q1)
    return {**{f: v.reshape(-1) for f, v in out.items()}, "score": score.reshape(-1)}


def exact(case, seed):
    path, R, S, K = case["path"], case["ranks"], case["steps"], case.get("kernels")
    if path == "iter_windows":
        return _exact_iter_windows(_step_times(case, seed), R, S)
    if path == "cross_rank":
        s = _summaries(case, seed)
        return _exact_cross_rank(s["count"], s["sum_ns"], R, S, K)
    if path == "l2":
        s = _summaries(case, seed)
        return _exact_l2(s["count"], s["sum_ns"], R, S, K, *_groups(R, K, case["tp"], case["pp"], case["ep"], seed))
    if path == "w1":
        return _exact_w1(_clusters(case, seed), R, S, K, case["grid"])
    if path != "pipeline":
        return None  # whole numbers and bytes only: compared value by value
    ev = _events(case, seed)
    off = ev["seg_off"]
    seg = torch.repeat_interleave(torch.arange(R * S, device=DEV), off[1:] - off[:-1])
    k, d = ev["kernel_id"].long(), ev["end_ns"] - ev["start_ns"]
    ok = (k >= 0) & (ev["stream"] >= 0) & (ev["stream"] < case["streams"]) & (d >= 0)
    cell, d, seg = (seg * K + k)[ok], d[ok], seg[ok]
    count = torch.bincount(cell, minlength=R * S * K)
    total = torch.zeros(R * S * K, dtype=torch.int64, device=DEV).index_add_(0, cell, d)
    last = torch.full((R * S,), I64_MIN, device=DEV).scatter_reduce(0, seg, ev["end_ns"][ok], "amax")
    first = torch.full((R * S,), I64_MAX, device=DEV).scatter_reduce(0, seg, ev["start_ns"][ok], "amin")
    y = torch.where(last >= first, last - first, 0)
    return {"sum": None, "xr": _exact_cross_rank(count, total, R, S, K), "l1": _exact_iter_windows(y, R, S), "kde": None,
            "w1": None, "l2": _exact_l2(count, total, R, S, K, *_groups(R, K, 2, 2, 2, seed)), "cp": None}
