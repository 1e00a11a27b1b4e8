"""The calls whose speed this framework is judged by, from the smallest to the largest.

A case is one pass of a program that uses the framework: a power trace (or the
readings of an energy counter) attributed to operator intervals, two systems
compared, a candidate sweep, a long trace streamed in chunks, or tensors turned
into their multi-mode SVD invariants.  Inputs are synthetic and made on the GPU
from the seed alone: every running sum is over whole ticks of time, so that the
same seed gives the same bits.
"""
from __future__ import annotations

import functools
import itertools
import math

import numpy as np
import torch

import paper_2512_08365_amd as mag

TICK = 1e-10  # seconds; interval bounds are whole numbers of it
TOP_K = 100


# ------------------------------------------------------------------- the cases

def _attr(name, n, rate, streams, per_stream, keys, zipf, median, **more):
    """One trace: n samples at `rate` Hz, `streams` x `per_stream` intervals
    (lognormal, median seconds), `keys` operator keys (Zipf exponent, 0: uniform)."""
    return {"name": name, "kind": "attribute", "n": n, "rate": rate, "streams": streams,
            "per_stream": per_stream, "keys": keys, "zipf": zipf, "median": median,
            "split": True, "latency": False, **more}


def listed():
    return [
        # a short profile looked at interactively: 10 s at 1 kHz, all arguments
        # left at their defaults; launches and host work are all there is
        _attr("attribute_short", 10_000, 1e3, 1, 2_000, 50, 1.1, 3e-3, capacity=0),
        # many concurrent streams of unequal length (a serving engine with
        # several worker streams): equal split among up to 16 intervals
        _attr("attribute_streams16", 20_000_000, 1e6, 16, 48_750, 5_000, 1.2, 200e-6,
              capacity=8_192, ragged=True),
        # operator windows of seconds over a bench meter's trace, odd sizes, full
        # power to each of three overlapping streams: intervals cross many tiles
        _attr("attribute_windows", 7_654_321, 1e5, 3, 333, 37, 0.0, 0.15, split=False,
              capacity=64),
        # the headline comparison: two 100 s traces at 1 MHz, four streams of a
        # million intervals each, both attributed and the top 100 keys ranked
        _attr("compare_streams4", 100_000_000, 1e6, 4, 1_000_000, 5_000, 1.2, 15e-6,
              kind="compare", capacity=5_632),
        # two decode-shaped traces (32 layers x 12 operators x 256 steps) with
        # latencies, and the detection of waste and trade-offs over them
        _attr("detect_decode", 2_000_000, 1e5, 1, 98_304, 416, 0.0, 20e-6 * 6, kind="detect",
              latency=True, capacity=512),
        # a baseline against eight candidates that ran the same operators: one
        # key plan, nine attributions, one batched comparison
        _attr("sweep_candidates8", 20_000_000, 2e5, 1, 1_000_000, 2_000, 0.0, 60e-6,
              kind="sweep", candidates=8, capacity=2_048),
        # an hour at 100 kHz that arrives in chunks of 32 M samples
        _attr("stream_hour", 360_000_000, 1e5, 1, 50_000_000, 20_000, 1.05, 40e-6,
              kind="stream", chunk=32_000_000, capacity=20_480),
        # a replay session read through a 50 Hz energy counter, with latencies
        {"name": "counter_session", "kind": "counter", "windows": 98_304, "keys": 416,
         "rate": 50.0, "replays": 1_000},
        # attention-shaped operator outputs: a batch of 64 tensors of rank 3
        {"name": "invariants_heads", "kind": "invariants", "shape": "32x128x128", "count": 64},
        # hidden states [batch, tokens, width] of a few layers: Gram sides of
        # hundreds, on both sides of the one-workgroup reduction's limit
        {"name": "invariants_hidden", "kind": "invariants", "shape": "4x512x768", "count": 4},
        # one square weight matrix
        {"name": "invariants_weight", "kind": "invariants", "shape": "4096x4096", "count": 1},
        # two systems' operator outputs of mixed ranks and odd sizes, invariants of
        # both and the matching of every pair
        {"name": "equivalence_mixed", "kind": "equivalence", "count": 48, "side": 40},
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    kind = rng.choice(["attribute", "attribute", "attribute", "compare", "detect", "sweep",
                       "stream", "counter", "invariants", "invariants", "invariants",
                       "equivalence"])
    if kind == "counter":
        return {"kind": kind, "windows": int(_log(rng, 500, 200_000)),
                "keys": int(_log(rng, 10, 4_000)), "rate": rng.choice([10.0, 20.0, 50.0]),
                "replays": int(_log(rng, 100, 2_000))}
    if kind == "equivalence":
        return {"kind": kind, "count": rng.randint(8, 64), "side": rng.randint(12, 64)}
    if kind == "invariants":
        rank = rng.choice([2, 2, 3, 3, 4])
        if rank == 2:
            a, b = _log(rng, 24, 3_000), _log(rng, 24, 4_096)
            count = rng.randint(1, 4) if min(a, b) < 1_500 else 1
            dims = [a, b]
        elif rank == 3:
            dims = [_log(rng, 2, 64), _log(rng, 48, 640), _log(rng, 32, 900)]
            count = rng.randint(1, 12)
        else:
            dims = [_log(rng, 1, 8), _log(rng, 4, 24), _log(rng, 16, 160), _log(rng, 16, 128)]
            count = rng.randint(1, 16)
        dims = [int(x) for x in dims]
        one = [(K, K * K * L) for K, L, _ in _spectra(dims)]
        # no more than the square weight matrix costs
        side, ops = sum(K for K, _ in one if K > 128), sum(f for _, f in one)
        count = max(1, min([count] + ([3_000 // side] if side else []) + [int(6e10 / ops)]))
        shape = "x".join(str(x) for x in dims)
        return {"kind": kind, "shape": shape, "count": count}
    streams = 1 if kind in ("sweep", "stream") else rng.choice([1, 1, 2, 3, 4, 6, 8, 16, 24])
    top = {"attribute": 4e7, "compare": 3e7, "detect": 8e6, "sweep": 8e6, "stream": 6e7}[kind]
    n = int(_log(rng, 3e3 if kind == "attribute" else 2e4, top))
    # samples per interval of one stream: about 7 in the hour-long trace, 25 to
    # 400 in the others, thousands in the windows
    per = _log(rng, 7.0, 1500.0)
    rate = rng.choice([1e3, 1e4, 1e5, 2e5, 1e6])
    per_stream = max(2, int(n / per))
    m = per_stream * streams
    keys = int(min(max(2, m // (40 if kind == "detect" else 2)), _log(rng, 10, 20_000)))
    case = _attr("", n, rate, streams, per_stream, keys, rng.choice([0.0, 1.05, 1.2]),
                 per / rate * rng.choice([0.15, 0.3, 0.5]), kind=kind,
                 capacity=keys + rng.randint(0, 64))
    del case["name"]
    if kind == "attribute":
        case["split"] = rng.random() < 0.75
        case["latency"] = rng.random() < 0.3
        case["ragged"] = rng.random() < 0.5
    elif kind == "detect":
        case["latency"] = True
    elif kind == "sweep":
        case["candidates"] = rng.randint(2, 9)
    elif kind == "stream":
        case["chunk"] = max(1_000, int(n / _log(rng, 2, 12)))
    return case


# ------------------------------------------------------------------ the inputs

def _gen(seed):
    g = torch.Generator("cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _rand(g, n):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _randn(g, n):
    return torch.randn(n, generator=g, device="cuda", dtype=torch.float64)


def _per_stream(case):
    """Intervals of each stream: equal, or falling to a third over the streams."""
    S, m = case["streams"], case["per_stream"]
    if not case.get("ragged") or S == 1:
        return [m] * S
    return [max(1, int(m * (1.0 - 0.66 * a / (S - 1)))) for a in range(S)]


def _keys(g, m, count, zipf):
    vocab = torch.randint(-2**63, 2**63 - 1, (count,), generator=g, device="cuda",
                          dtype=torch.int64)
    if zipf:
        w = np.arange(1, count + 1, dtype=np.float64) ** -zipf
        cdf = torch.from_numpy(np.cumsum(w / w.sum())).cuda()
        idx = torch.searchsorted(cdf, _rand(g, m)).clamp_(max=count - 1)
    else:
        idx = torch.randint(0, count, (m,), generator=g, device="cuda", dtype=torch.int64)
    # every operator runs at least once
    idx[torch.randperm(m, generator=g, device="cuda")[:count]] = torch.arange(
        min(m, count), device="cuda")
    return vocab[idx], idx


def _times(g, case):
    """Sample times with 5 % jitter."""
    t = torch.arange(case["n"], device="cuda", dtype=torch.float64)
    t += (_rand(g, case["n"]) - 0.5) * 0.1
    return t.div_(case["rate"])


def _intervals(g, case):
    """Interval bounds of every stream: lognormal lengths (sigma 1) and
    exponential gaps that together span the trace (a few reach past its end)."""
    span = case["n"] / case["rate"]
    ss, ee, off = [], [], [0]
    for m in _per_stream(case):
        mean = case["median"] * math.exp(0.5)
        scale = min(1.0, 0.95 * span / (m * mean))  # lengths alone must fit the trace
        gap = max(span / m - mean * scale, 0.0)
        dur = torch.exp(_randn(g, m)) * (case["median"] * scale / TICK)
        gaps = torch.log(_rand(g, m).clamp_(min=1e-12)) * (-gap / TICK)
        cuts = torch.stack([gaps, dur], 1).round_().clamp_(min=1.0).to(torch.int64).reshape(-1)
        del dur, gaps
        cuts = torch.cumsum(cuts, 0).to(torch.float64) * TICK
        ss.append(cuts[0::2])
        ee.append(cuts[1::2])
        off.append(off[-1] + m)
    return torch.cat(ss).contiguous(), torch.cat(ee).contiguous(), off


def _power(g, case, t, s, e, idx, off, levels):
    """Idle power, the level of each active interval's key, and sensor noise."""
    P = torch.randn(case["n"], generator=g, device="cuda", dtype=torch.float32)
    # (a meter that averages over its sampling period: little noise where keys
    # are judged against a threshold)
    P.mul_(1.0 if case["kind"] == "detect" else 20.0).add_(100.0)
    step = 1 << 26
    for a in range(len(off) - 1):
        sa, ea, ka = s[off[a]:off[a + 1]], e[off[a]:off[a + 1]], idx[off[a]:off[a + 1]]
        for lo in range(0, case["n"], step):
            x = t[lo:lo + step]
            at = torch.searchsorted(sa, x, right=True).sub_(1).clamp_(min=0)
            on = (x >= sa[at]) & (x < ea[at])
            P[lo:lo + step] += torch.where(on, levels[ka[at]], torch.zeros_like(levels[:1]))
    return P.clamp_(min=0.0)


def _levels(g, case):
    return 50.0 + 110.0 * torch.rand(case["keys"], generator=g, device="cuda",
                                     dtype=torch.float32)


def _sides(case, seed, count):
    """`count` traces of the same operators: the others' keys draw 0.8 to 1.5
    times the first's power, or, where inefficiencies are detected, the same
    power but for every fourth key, which draws 2.5 times as much."""
    g = _gen(seed)
    t = _times(g, case)
    s, e, off = _intervals(g, case)
    keys, idx = _keys(g, int(s.shape[0]), case["keys"], case["zipf"])
    base = _levels(g, case)
    P = []
    for c in range(count):
        f = 0.8 + 0.7 * torch.rand(case["keys"], generator=g, device="cuda", dtype=torch.float32)
        if case["kind"] == "detect":
            f = 1.0 + 1.5 * (torch.arange(case["keys"], device="cuda") % 4 == 0)
        P.append(_power(g, case, t, s, e, idx, off, base * f if c else base))
    return t, P, s, e, keys, off


def _counter_inputs(case, seed):
    g = _gen(seed)
    m, reps = case["windows"], case["replays"]
    dur = torch.exp(_randn(g, m)) * (20e-6 * reps / TICK)
    pause = (0.010 + 0.040 * _rand(g, m)) / TICK
    cuts = torch.stack([pause, dur], 1).round_().clamp_(min=1.0).to(torch.int64).reshape(-1)
    cuts = torch.cumsum(cuts, 0).to(torch.float64) * TICK
    s, e = cuts[0::2].contiguous(), cuts[1::2].contiguous()
    span = m * (0.030 + 20e-6 * reps * math.exp(0.5)) * 1.1 + 1.0
    n = int(span * case["rate"]) + 2
    delay = 0.1
    t = torch.arange(n, device="cuda", dtype=torch.float64)
    t = (t + (_rand(g, n) - 0.5) * 0.1) / case["rate"] - 0.5 + delay
    watts = 400.0 + 250.0 * torch.sin(torch.arange(n - 1, device="cuda", dtype=torch.float64) / 97.0)
    uj = ((watts + 40.0 * (_rand(g, n - 1) - 0.5)) / case["rate"] * 1e6).round_().to(torch.int64)
    C = torch.full((n,), 5e5, device="cuda", dtype=torch.float64)
    C[1:] += torch.cumsum(uj, 0).to(torch.float64) * 1e-6
    keys, _ = _keys(g, m, case["keys"], 0.0)
    replays = torch.full((m,), reps, device="cuda", dtype=torch.int32)
    return t, C, delay, s, e, replays, keys


def _dims(case):
    return tuple(int(x) for x in case["shape"].split("x"))


def _tensor(g, shape):
    """An activation-like tensor: normal entries, with a gain for every index of
    every mode (fp32)."""
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    for d, size in enumerate(shape):
        w = torch.randn(size, generator=g, device="cuda", dtype=torch.float32)
        x *= torch.exp(0.5 * w).reshape([-1 if i == d else 1 for i in range(len(shape))])
    return x


def _mixed_shapes(case):
    """Odd shapes of ranks 1 to 5 (the same for every seed)."""
    top = case["side"]
    ranks = itertools.cycle([2, 3, 1, 4, 3, 2, 5])
    out, a = [], 3
    for _ in range(case["count"]):
        r = next(ranks)
        shape = []
        for i in range(r):
            a = (a * 37 + 11) % 1009
            hi = top * 3 if r == 2 else top if r == 3 else max(2, top // 4) if r == 4 else max(2, top // 8)
            shape.append((1_000 if r == 1 else 2) + a % (top * 8 if r == 1 else hi))
        out.append(tuple(shape))
    return out


def _equivalence_inputs(case, seed):
    """Set A, and set B: A's tensors in another order, every other one with its
    modes permuted (equivalent), the rest drawn anew (not equivalent)."""
    g = _gen(seed)
    shapes = _mixed_shapes(case)
    a = [_tensor(g, sh) for sh in shapes]
    b = []
    for i in range(len(a)):
        src = a[(i * 5 + 2) % len(a)]
        if i % 2 == 0:
            b.append(src.permute(*reversed(range(src.dim()))).contiguous())
        else:
            b.append(_tensor(g, tuple(src.shape)))
    return a, b


@functools.lru_cache(maxsize=None)
def _side_stream():
    """The second stream of a program that compares two systems."""
    return torch.cuda.Stream()


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "counter":
        st["in"] = _counter_inputs(case, seed)
        return st
    if kind == "invariants":
        g = _gen(seed)
        st["tensors"] = [_tensor(g, _dims(case)) for _ in range(case["count"])]
        return st
    if kind == "equivalence":
        st["a"], st["b"] = _equivalence_inputs(case, seed)
        return st
    count = 2 if kind in ("compare", "detect") else 1 + case.get("candidates", 0)
    t, P, s, e, keys, off = _sides(case, seed, count)
    st.update(t=t, P=P, s=s, e=e, keys=keys, off=off)
    m, cap = int(s.shape[0]), case["capacity"]
    if kind in ("compare", "detect", "sweep"):
        # a program that attributes again and again keeps its workspaces
        plan = mag.KeyPlan(keys, cap) if kind == "sweep" else None
        st["plan"] = plan
        flags = mag.EQUAL_SPLIT | (mag.KEY_LATENCY if case["latency"] else 0)
        size = mag.workspace_size(case["n"], m, cap, case["streams"], off, flags, plan)
        st["work"] = [torch.empty(size, dtype=torch.uint8, device="cuda") for _ in range(count)]
    if kind == "compare":
        st["side"] = _side_stream()
    if kind == "stream":
        c = case["chunk"]
        st["chunks"] = [(t[i:i + c], P[0][i:i + c]) for i in range(0, case["n"], c)]
    return st


# -------------------------------------------------------------------- one pass

def _attribute(st, side, **more):
    case = st["case"]
    return mag.attribute(st["t"], st["P"][side], st["s"], st["e"], st["keys"],
                         n_streams=case["streams"], stream_offsets=st["off"],
                         equal_split=case["split"], latency=case["latency"],
                         key_capacity=case["capacity"] or None, **more)


def run(state):
    st = state
    case = st["case"]
    kind = case["kind"]
    if kind == "attribute":
        return _attribute(st, 0)
    if kind == "compare":
        # both sides enqueued, the second on a stream of its own behind the
        # first's trace integration, and one wait for each
        done = torch.cuda.Event()
        here = torch.cuda.current_stream()
        a = _attribute(st, 0, workspace=st["work"][0], asynchronous=True, tiles_done=done)
        with torch.cuda.stream(st["side"]):
            b = _attribute(st, 1, workspace=st["work"][1], asynchronous=True, tiles_wait=done)
        a, b = a.finish(), b.finish()
        for x in itertools.chain(b[0].values(), b[1].values()):
            x.record_stream(here)
        return a, b, mag.diff(a[1], b[1], TOP_K)
    if kind == "detect":
        a = _attribute(st, 0, workspace=st["work"][0], asynchronous=True)
        b = _attribute(st, 1, workspace=st["work"][1], asynchronous=True)
        a, b = a.finish(), b.finish()
        return a, b, mag.detect(a[1], b[1])
    if kind == "sweep":
        wait = [_attribute(st, c, workspace=st["work"][c], asynchronous=True,
                           key_plan=st["plan"]) for c in range(len(st["P"]))]
        done = [w.finish() for w in wait]
        ranks = mag.diff_batch(done[0][1], [d[1] for d in done[1:]], TOP_K)
        # the baseline whole; of each candidate its energies and its ranking
        return done[0], [(d[0]["energy"], r["key"], r["ratio"], r["energy_a"], r["energy_b"])
                         for d, r in zip(done[1:], ranks)]
    if kind == "stream":
        h = mag.Stream(case["n"], st["s"], st["e"], st["keys"], n_streams=case["streams"],
                       stream_offsets=st["off"], equal_split=case["split"],
                       key_capacity=case["capacity"])
        for t, P in st["chunks"]:
            h.push(t, P)
        return h.end()
    if kind == "counter":
        t, C, delay, s, e, replays, keys = st["in"]
        pi, pk, summ = mag.attribute_counter(t, C, s, e, keys, delay=delay, replays=replays,
                                             latency=True)
        return pi, pk, {k: v for k, v in summ.items() if not k.endswith("_ms")}
    if kind == "invariants":
        return mag.invariants(st["tensors"])[0]
    sa, _ = mag.invariants(st["a"])
    sb, _ = mag.invariants(st["b"])
    return sa, sb, mag.match(st["a"], sa, st["b"], sb)


# --------------------------------------------------- what a pass cannot do without

def _spectra(shape):
    """(K, L) of every unfolding whose mode subset holds mode 0."""
    r = len(shape)
    for bits in range(1, (1 << r) - 1, 2):
        M = math.prod(n for i, n in enumerate(shape) if bits >> i & 1)
        N = math.prod(n for i, n in enumerate(shape) if not bits >> i & 1)
        yield min(M, N), max(M, N), bits


def _invariants_work(shapes):
    # fp32 elements in, fp64 spectra out; the products of one triangle of the Gram
    # matrix and its reduction to tridiagonal form
    b = f = 0
    for sh in shapes:
        b += 4 * math.prod(sh)
        for K, L, _ in _spectra(sh):
            b += 8 * K
            f += K * (K + 1) * L + 4 * K ** 3 // 3
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "invariants":
        b, f = _invariants_work([_dims(case)] * case["count"])
        return {"bytes": b, "flops": f}
    if kind == "equivalence":
        b, f = _invariants_work(2 * _mixed_shapes(case))
        return {"bytes": b + case["count"] ** 2, "flops": f}
    if kind == "counter":
        m = case["windows"]
        n = (m * (0.030 + 20e-6 * case["replays"] * math.exp(0.5)) * 1.1 + 1.0) * case["rate"]
        return {"bytes": 16 * n + 52 * m + 40 * case["keys"], "flops": 12 * m}
    n, m, K = case["n"], sum(_per_stream(case)), min(case["keys"], sum(_per_stream(case)))
    row = 32 + (8 if case["latency"] else 0)
    one = 12 * n + 48 * m + row * K  # samples, intervals and their outputs, key rows
    ops = 5 * n + 20 * m
    sides = 2 if kind in ("compare", "detect") else 1 + case.get("candidates", 0)
    # (sides that share sample times, bounds and keys are still traces of their own)
    return {"bytes": sides * one + (sides - 1) * 48 * min(K, TOP_K), "flops": sides * ops}


def tolerance(case):
    # Singular values are square roots of eigenvalues that are exact to about
    # 1e-15 of the largest, so a value far below the largest is the less exact
    # the smaller it is: 8e-11 and 5e-9 measured on a square matrix against a
    # singular value decomposition, with a spread of ten between seeds (its
    # smallest singular value decides), 1e-13 and 1e-11 on other shapes.
    if case["kind"] in ("invariants", "equivalence"):
        return {"rel": 1e-9, "max": 1e-7}
    # Sums of up to a million doubles: 2.3e-13 (the idle energy of a crowded
    # trace) and 7.1e-13 (single intervals) measured against extended precision.
    return {"rel": 1e-12, "max": 3e-12}


# ------------------------------------------------------------ the answer in 64 bits

def _np(x):
    return x.cpu().numpy()


def _integral(t, P):
    """x -> integral of the interpolated power from t[0] to x (x inside the trace)."""
    h = np.diff(t).astype(np.longdouble)
    cum = np.zeros(len(t), np.longdouble)
    np.cumsum((P[:-1] + P[1:]) * h / 2, out=cum[1:])

    def F(x):
        j = np.clip(np.searchsorted(t, x, side="right") - 1, 0, len(t) - 2)
        d = x.astype(np.longdouble) - t[j]
        return cum[j] + d * (P[j] + (P[j + 1] - P[j]) / h[j] * d / 2)

    return F, cum[-1]


def _energies(t, P, s, e, split):
    P = P.astype(np.float64)
    F, total = _integral(t, P)
    m = len(s)
    x = np.clip(np.concatenate([s, e]), t[0], t[-1])
    order = np.argsort(x, kind="stable")
    Fx = F(x[order])
    active = np.cumsum(np.where(order < m, 1, -1))
    gap = np.diff(Fx, append=total)
    G = np.zeros(2 * m + 1, np.longdouble)
    np.cumsum(np.where(active > 0, gap / np.maximum(active, 1) if split else gap, 0), out=G[1:])
    at = np.empty(2 * m, np.int64)
    at[order] = np.arange(2 * m)
    idle = Fx[0] + gap[active == 0].sum()
    E = G[at[m:]] - G[at[:m]] if split else F(x[m:]) - F(x[:m])
    return E, total, idle


def _table(keys, E, dur=None):
    u = keys.view(np.uint64)
    order = np.argsort(u, kind="stable")
    first = np.flatnonzero(np.concatenate([[True], np.diff(u[order]) != 0]))
    count = np.diff(np.append(first, len(u)))
    total = np.add.reduceat(E[order], first)
    dev = E[order] - np.repeat(total / count, count)
    out = {"keys": None, "count": None, "sum": total.astype(np.float64),
           "m2": np.add.reduceat(dev * dev, first).astype(np.float64)}
    if dur is not None:
        out["duration"] = np.add.reduceat(dur[order], first).astype(np.float64)
    return out, u[order][first], total


def _exact_attribute(t, P, s, e, keys, case):
    E, total, idle = _energies(t, P, s, e, case["split"])
    dur = e.astype(np.longdouble) - s if case["latency"] else None
    tab, uniq, sums = _table(keys, E, dur)
    summ = {"trace_energy": float(total), "idle_energy": float(idle),
            "attributed_energy": float(E.sum()), "n_clipped": None, "n_keys": None}
    return ({"energy": E.astype(np.float64), "start_idx": None, "end_idx": None}, tab, summ), sums, uniq


def _rank(a, b, uniq, k):
    # (a key whose intervals lie past the trace's end has no energy on either side)
    r = np.where(a > 0, (b - a) / np.where(a > 0, a, 1), 0)
    order = np.lexsort((uniq, -r))[:k]
    return order, r[order].astype(np.float64)


def _singular_values(x):
    x = _np(x).astype(np.float64)
    out = []
    for K, _, bits in _spectra(x.shape):
        rows = [i for i in range(x.ndim) if bits >> i & 1]
        cols = [i for i in range(x.ndim) if not bits >> i & 1]
        M = math.prod(x.shape[i] for i in rows)
        out.append(np.linalg.svd(x.transpose(rows + cols).reshape(M, -1), compute_uv=False))
    return out


def _all_spectra(tensors):
    out = [v for x in tensors for v in _singular_values(x)]
    return np.concatenate(out) if out else np.zeros(0)


def exact(case, seed):
    kind = case["kind"]
    if kind == "invariants":
        # (a singular value decomposition of sides K and L: about 4 L K^2 operations)
        if case["count"] * sum(L * K * K for K, L, _ in _spectra(_dims(case))) > 8e10:
            return None
        g = _gen(seed)
        return _all_spectra([_tensor(g, _dims(case)) for _ in range(case["count"])])
    if kind == "equivalence":
        a, b = _equivalence_inputs(case, seed)
        return _all_spectra(a), _all_spectra(b), None
    if kind == "counter":
        t, C, delay, s, e, replays, keys = _counter_inputs(case, seed)
        t, C, s, e, reps, keys = map(_np, (t, C, s, e, replays, keys))
        u = t - delay

        def at(x):
            j = np.clip(np.searchsorted(u, x, side="right") - 1, 0, len(u) - 2)
            w = (np.clip(x, u[0], u[-1]).astype(np.longdouble) - u[j]) / (u[j + 1] - u[j]).astype(np.longdouble)
            return C[j] + w * (C[j + 1].astype(np.longdouble) - C[j])

        inc = at(e) - at(s)
        E = inc / reps
        tab, _, _ = _table(keys, E, (e.astype(np.longdouble) - s) / reps)
        return ({"energy": E.astype(np.float64), "start_idx": None, "end_idx": None}, tab,
                {"trace_energy": float(C[-1] - C[0]), "idle_energy": None,
                 "attributed_energy": float(E.sum()), "n_clipped": None, "n_keys": None})
    count = 2 if kind in ("compare", "detect") else 1 + case.get("candidates", 0)
    if count * (case["n"] + 6 * sum(_per_stream(case))) > 60e6:
        return None
    t, P, s, e, keys, _ = _sides(case, seed, count)
    t, s, e, keys = map(_np, (t, s, e, keys))
    got = [_exact_attribute(t, _np(p), s, e, keys, case) for p in P]
    if kind in ("attribute", "stream"):
        return got[0][0]
    uniq = got[0][2]
    if kind == "sweep":
        ranks = [_rank(got[0][1], g[1], uniq, TOP_K) for g in got[1:]]
        return got[0][0], [(g[0][0]["energy"], None, r, got[0][1][o].astype(np.float64),
                            g[1][o].astype(np.float64)) for g, (o, r) in zip(got[1:], ranks)]
    ea, eb = got[0][1], got[1][1]
    order, r = _rank(ea, eb, uniq, TOP_K if kind == "compare" else len(uniq))
    if kind == "detect":
        order, r = order[r >= 0.10], r[r >= 0.10]
    rank = {"ratio": r, "energy_a": ea[order].astype(np.float64),
            "energy_b": eb[order].astype(np.float64)}
    if kind == "detect":
        rank["latency_a"] = got[0][0][1]["duration"][order]
        rank["latency_b"] = got[1][0][1]["duration"][order]
    return got[0][0], got[1][0], rank
