"""Parity of the counter (software replay) attribution, through the C ABI,
with the CPU oracle.

Sample indices, key grouping and counts are bit-exact; window energies within
1e-9 relative; the summary's totals within 1e-12 of the counter's whole
increase.  Cases span many 64-window chunks and 256-reading blocks with ragged
tails, windows that reach past the readings, bounds exactly on shifted reading
times, zero-length windows, flat counter stretches, delays of either sign,
irregular reading spacing (the chunk-boundary search's fallback), and every
device-detected input error.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_energy_close, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2512_08365_amd as mag
    mag.version()
    yield


def _dev(c):
    import torch
    d = {k: torch.from_numpy(np.ascontiguousarray(c[k], np.float64)).cuda()
         for k in ("t", "C", "s", "e")}
    d["key"] = torch.from_numpy(np.ascontiguousarray(c["key"], np.uint64).view(np.int64)).cuda()
    d["reps"] = None if c["reps"] is None else torch.from_numpy(
        np.ascontiguousarray(c["reps"], np.int32)).cuda()
    return d


def compare(c, label, group=True, validate=True):
    import paper_2512_08365_amd as mag
    log(f"[counter] {label}: n={len(c['t'])} m={len(c['s'])} delay={c['delay']}")
    d = _dev(c)
    pi, pk, summ = mag.attribute_counter(d["t"], d["C"], d["s"], d["e"],
                                         d["key"] if group else None, delay=c["delay"],
                                         replays=d["reps"], validate=validate)
    ref = oracle.counter_attribute(c["t"], c["C"], c["s"], c["e"], delay=c["delay"],
                                   reps=c["reps"])
    assert np.array_equal(pi["start_idx"].cpu().numpy(), ref["start_idx"]), label
    assert np.array_equal(pi["end_idx"].cpu().numpy(), ref["end_idx"]), label
    assert_energy_close(pi["energy"].cpu().numpy(), ref["energy"], f"{label} energy")
    scale = abs(ref["trace_energy"]) + 1e-300
    assert summ["trace_energy"] == ref["trace_energy"], label
    assert abs(summ["idle_energy"] - ref["idle_energy"]) <= 1e-12 * scale, label
    assert abs(summ["attributed_energy"] - ref["attributed_energy"]) <= \
        1e-12 * scale + 1e-9 * abs(ref["attributed_energy"]), label
    assert summ["n_clipped"] == ref["n_clipped"], label
    if group and len(c["s"]):
        g = oracle.groupby(c["key"], ref["energy"])
        assert np.array_equal(pk["keys"].cpu().numpy().view(np.uint64), g["keys"]), label
        assert np.array_equal(pk["count"].cpu().numpy(), g["count"]), label
        assert_energy_close(pk["sum"].cpu().numpy(), g["sum"], f"{label} key sums")
        second = g["m2"] + g["sum"] ** 2 / np.maximum(g["count"], 1)
        assert np.all(np.abs(pk["m2"].cpu().numpy() - g["m2"]) <= 1e-9 * second), label
    return pi, pk, summ


def test_tiny_fuzz():
    for seed in range(60):
        n = 2 + (seed * 53) % 400
        m = (seed * 29) % 150
        c = synth.counter_case(7000 + seed, n=n, m=m, replays=bool(seed % 3),
                               outside=bool(seed % 4), zero_len=0.1 * (seed % 2))
        compare(c, f"tiny seed{seed}", group=bool(seed % 5))


@pytest.mark.parametrize("n,m", [(2, 0), (2, 1), (3, 64), (257, 64), (256, 65), (5000, 63),
                                 (20000, 129), (300, 5000), (70000, 6400)])
def test_chunk_and_block_edges(n, m):
    c = synth.counter_case(n * 31 + m, n=n, m=m)
    compare(c, f"edges n={n} m={m}")


def test_dense_windows_in_one_segment():
    # many windows between two readings: every endpoint in the same segment
    c = synth.counter_case(11, n=40, m=3000, outside=False, snap=0.0)
    compare(c, "dense")


def test_sparse_windows_over_long_readings():
    # few windows, each chunk streams tens of thousands of readings
    c = synth.counter_case(12, n=200_000, m=150, period=0.001)
    compare(c, "sparse")


def test_irregular_reading_spacing():
    for seed in range(4):
        c = synth.counter_case(13 + seed, n=50_000, m=4000, irregular=True)
        compare(c, f"irregular seed{seed}")


@pytest.mark.parametrize("delay", [0.0, 0.25, -0.07, 1e6])
def test_delays(delay):
    c = synth.counter_case(21, n=3000, m=700, delay=delay)
    compare(c, f"delay {delay}")


def test_replay_session_full_size():
    c = synth.replay_session(0)
    pi, pk, summ = compare(c, "replay session")
    assert summ["n_keys"] == len(np.unique(c["key"]))


def test_skip_validate_gives_the_same_result():
    c = synth.counter_case(31, n=5000, m=900)
    a = compare(c, "validated")
    b = compare(c, "unvalidated", validate=False)
    assert np.array_equal(a[0]["energy"].cpu().numpy(), b[0]["energy"].cpu().numpy())


@pytest.mark.parametrize("case,code", [
    ("t_not_increasing", -5), ("t_nan", -5), ("shift_collapses", -5), ("delay_inf", -5),
    ("counter_decreases", -13), ("counter_nan", -13),
    ("start_after_end", -7), ("overlap", -7), ("zero_replays", -7), ("bound_nan", -7),
])
def test_device_detected_errors(case, code):
    import torch
    import paper_2512_08365_amd as mag
    rng = np.random.default_rng(5)
    c = synth.counter_case(41, n=3000, m=400, delay=0.0, zero_len=0.0)
    t, C, s, e, reps = (c["t"].copy(), c["C"].copy(), c["s"].copy(), c["e"].copy(),
                        c["reps"].copy())
    delay = 0.0
    j = int(rng.integers(1, 2999))
    i = int(rng.integers(1, 399))
    if case == "t_not_increasing":
        t[j] = t[j - 1]
    elif case == "t_nan":
        t[j] = np.nan
    elif case == "shift_collapses":
        t = np.arange(3000, dtype=np.float64) * 1e-300
        delay = 1.0
    elif case == "delay_inf":
        delay = np.inf
    elif case == "counter_decreases":
        C[j] = C[j - 1] - 1.0
    elif case == "counter_nan":
        C[j] = np.nan
    elif case == "start_after_end":
        s[i] = e[i] + 1e-9
        e[i - 1] = min(e[i - 1], s[i])
    elif case == "overlap":
        s[i] = e[i - 1] - 1e-6
    elif case == "zero_replays":
        reps[i] = 0
    elif case == "bound_nan":
        e[i] = np.nan
    with pytest.raises(oracle.OracleError) as want:
        oracle.counter_attribute(t, C, s, e, delay=delay, reps=reps)
    assert want.value.code == code
    d = {k: torch.from_numpy(v).cuda() for k, v in (("t", t), ("C", C), ("s", s), ("e", e))}
    with pytest.raises(mag.MagnetonError) as got:
        mag.attribute_counter(d["t"], d["C"], d["s"], d["e"], delay=delay,
                              replays=torch.from_numpy(reps).cuda())
    assert got.value.code == code, case


def test_asynchronous_and_timed_calls_equal_the_synchronous_one():
    import paper_2512_08365_amd as mag
    c = synth.counter_case(51, n=20000, m=3000)
    d = _dev(c)
    args = (d["t"], d["C"], d["s"], d["e"], d["key"])
    kw = dict(delay=c["delay"], replays=d["reps"], latency=True)
    ref = mag.attribute_counter(*args, **kw)
    pend = mag.attribute_counter(*args, asynchronous=True, time_kernels=True, **kw)
    got = pend.finish()
    for k in ("energy", "start_idx", "end_idx"):
        assert np.array_equal(got[0][k].cpu().numpy(), ref[0][k].cpu().numpy()), k
    for k in ("keys", "count"):
        assert np.array_equal(got[1][k].cpu().numpy(), ref[1][k].cpu().numpy()), k
    assert_energy_close(got[1]["duration"].cpu().numpy(), ref[1]["duration"].cpu().numpy(),
                        "latency")
    assert got[2]["n_clipped"] == ref[2]["n_clipped"]
    assert got[2]["kernel_ms"] > 0.0 and got[2]["device_ms"] >= got[2]["kernel_ms"]


# windows so far apart that a chunk of 64 spans more than the 4,096 readings it
# would stream (each endpoint is then searched in memory), spans around that
# limit, readings long before the first and after the last window, and the
# edges of the pieces in which readings are checked (2,048)
@pytest.mark.parametrize("n,m", [(4096, 40), (4097, 40), (4200, 64), (5000, 64), (60000, 3),
                                 (100_000, 150), (2047, 5), (2048, 5), (2049, 5), (6145, 1)])
def test_sparse_windows_and_unwatched_readings(n, m):
    c = synth.counter_case(8100 + n + m, n=n, m=m, outside=n % 2 == 0)
    compare(c, f"sparse n{n} m{m}")
    c = synth.counter_case(8200 + n + m, n=n, m=m, irregular=True)
    compare(c, f"sparse irregular n{n} m{m}")
    # every window inside a short stretch: most readings lie outside it
    c = synth.counter_case(8300 + n + m, n=n, m=m, outside=False)
    lo, span = c["t"][0], c["t"][-1] - c["t"][0]
    for k in ("s", "e"):
        c[k] = lo + 0.4 * span + (c[k] - lo) * 0.01
    compare(c, f"clustered n{n} m{m}")


@pytest.mark.parametrize("j", [0, 1, 2047, 2048, 5999])
def test_bad_reading_anywhere(j):
    """A reading far from every window is checked all the same."""
    import paper_2512_08365_amd as mag
    c = synth.counter_case(8400, n=6000, m=4, outside=False, delay=0.0)
    for name, value, code in (("C", np.nan, -13), ("t", np.nan, -5)):
        d = {k: np.array(c[k]) for k in c if isinstance(c[k], np.ndarray)}
        d["reps"] = c["reps"]
        d[name][j] = value
        g = _dev(d)
        with pytest.raises(mag.MagnetonError) as err:
            mag.attribute_counter(g["t"], g["C"], g["s"], g["e"], g["key"], replays=g["reps"])
        assert err.value.code in ((code,) if name == "C" else (code, -7)), (name, j)


def _session(kind):
    """(readings, window starts and ends): windows dense in the middle of the
    readings; far apart; two dense stretches with a long pause; one; none."""
    rng = np.random.default_rng(8500)
    n = {"dense": 4000, "apart": 60_000, "pause": 30_000, "one": 9000, "none": 5000}[kind]
    t = np.arange(n) * 0.02 + rng.uniform(0.0, 0.01, n)

    def windows(lo, hi, m):
        cuts = np.sort(rng.uniform(t[lo], t[hi], 2 * m))
        return cuts[0::2], cuts[1::2]

    parts = {"dense": [(1000, 3000, 1500)], "apart": [(5000, 55_000, 150)],
             "pause": [(3000, 4000, 200), (25_000, 26_000, 300)], "one": [(4000, 4500, 1)],
             "none": []}[kind]
    ws = [windows(*x) for x in parts] or [(np.zeros(0), np.zeros(0))]
    return t, np.concatenate([w[0] for w in ws]), np.concatenate([w[1] for w in ws])


@pytest.mark.parametrize("kind", ["dense", "apart", "pause", "one", "none"])
def test_every_reading_is_checked(kind):
    """One bad reading (a time that does not rise, a counter that falls) at a time:
    at the trace's ends, around the first reading of every chunk of windows and
    the last window's last one, at the edges of the checked pieces, and anywhere."""
    import torch
    import paper_2512_08365_amd as mag
    t, s, e = _session(kind)
    n, m = len(t), len(s)
    rng = np.random.default_rng(n)
    C = np.cumsum(rng.uniform(0.5, 1.5, n))
    edges = list(np.searchsorted(t, s[::64])) + list(np.searchsorted(t, e[-1:]))
    at = {1, 2, n - 2, n - 1} | {int(x + o) for x in edges for o in (-1, 0, 1)} \
        | {int(x + o) for x in edges[-1:] + edges[:1] for o in (2047, 2048, 2049)} \
        | {int(x) for x in rng.integers(1, n, 30)}
    d = {k: torch.from_numpy(v).cuda() for k, v in (("t", t), ("C", C), ("s", s), ("e", e))}
    key = torch.zeros(m, dtype=torch.int64, device="cuda") if m else None
    log(f"[counter] every reading: {kind} n={n} m={m} places={len(at)}")

    def call():
        return mag.attribute_counter(d["t"], d["C"], d["s"], d["e"], key, key_capacity=4)

    call()
    for j in sorted(x for x in at if 0 < x < n):
        for name, value, code in (("t", t[j - 1], -5), ("C", C[j - 1] - 1e-6, -13)):
            keep = float(d[name][j])
            d[name][j] = value
            with pytest.raises(mag.MagnetonError) as err:
                call()
            assert err.value.code == code, (kind, name, j)
            d[name][j] = keep
    call()
