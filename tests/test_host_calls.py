"""What the library asks of the HIP runtime, in which order, and what it does
when the runtime refuses: the library's host code runs in a child process over a
stand-in runtime (hip_double.c) that records its calls, so no GPU is needed and
no kernel runs."""
import ctypes
import importlib.util
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def double(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("double") / "hip_double.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", "-o", so,
                           os.path.join(HERE, "hip_double.c")])
    return so


def _run(double, name):
    """One of the functions below, in a process of its own (the library keeps
    records per thread, so each starts from none)."""
    env = dict(os.environ)
    env["LD_PRELOAD"] = " ".join(x for x in (env.get("LD_PRELOAD"), double) if x)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), name], env=env,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


# ------------------------------------------------------------ in the child

class Library:
    def __init__(self):
        spec = importlib.util.spec_from_file_location(
            "native", os.path.join(ROOT, "paper_2512_08365_amd", "_native.py"))
        self.N = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.N)
        self.lib = self.N.load()
        self.d = ctypes.CDLL(None)
        self.d.double_log.restype = ctypes.c_char_p
        self.next_ws = 1 << 32

    def log(self):
        return self.d.double_log().decode().splitlines()

    def clear(self):
        self.d.double_clear()

    def fail(self, name, times=1, after=0):
        self.d.double_fail(name.encode(), times, after)

    def ws(self):
        """A workspace that no call has used (never followed)."""
        self.next_ws += 1 << 30
        return self.next_ws

    def ok(self, rc):
        assert rc == 0, (rc, self.lib.mag_last_error())

    def stats(self, cap):
        s = self.N.KeyStats()
        s.sum = s.m2 = s.count = 4096
        s.capacity = s.n_keys = cap
        return s

    def attribute(self, ws, m=10_000, flags=0):
        N = self.N
        o = N.AttrOpts(1, flags | N.MAG_EQUAL_SPLIT, None)
        return self.lib.mag_attribute(4096, 4096, 100_000, 4096, 4096, 4096, m, ctypes.byref(o), None,
                                      4096, ctypes.byref(self.stats(64)), None, ws, 1 << 29, None)

    def counter(self, ws):
        return self.lib.mag_attribute_counter(4096, 4096, 5_000, 0.1, 4096, 4096, None, 4096, 10_000, 0,
                                              None, 4096, ctypes.byref(self.stats(64)), None, ws,
                                              1 << 29, None)

    def rank_out(self):
        r = self.N.RankOut()
        r.key = r.ratio = r.energy_a = r.energy_b = r.count_a = r.count_b = 4096
        r.capacity = 10
        return r

    def diff(self, ws):
        a, b = self.stats(64), self.stats(64)
        return self.lib.mag_diff(4096, ctypes.byref(a), 4096, ctypes.byref(b), 10,
                                 ctypes.byref(self.rank_out()), ws, 1 << 29, None)

    def stream(self, ws, n=5_000):
        N = self.N
        h = ctypes.c_void_p()
        o = N.AttrOpts(1, N.MAG_EQUAL_SPLIT, None)
        self.ok(self.lib.mag_stream_begin(ctypes.byref(h), n, 4096, 4096, 4096, 10_000,
                                          ctypes.byref(o), None, 64, ws, 1 << 29, None))
        return h

    def streamed(self, ws):
        h = self.stream(ws)
        self.ok(self.lib.mag_stream_push(h, 4096, 4096, 5_000))
        return self.lib.mag_stream_end(h, 4096, ctypes.byref(self.stats(64)), None)


    def invariants(self, shapes, ws=None):
        """fp32 tensors of these shapes (never followed)"""
        N = self.N
        ts = (N.Tensor * len(shapes))()
        for t, sh in zip(ts, shapes):
            t.data, t.rank = 1 << 20, len(sh)
            for i, x in enumerate(sh):
                t.dims[i] = x
        b = ctypes.c_size_t(0)
        self.ok(self.lib.mag_invariants_workspace_size(ts, len(shapes), ctypes.byref(b)))
        return self.lib.mag_invariants(ts, len(shapes), 1 << 20, ws or self.ws(), b.value, None)


def first(log, what):
    return next((i for i, x in enumerate(log) if re.search(what, x)), len(log))


def status_record_waits_for_the_launches():
    """A call's record of its workspace costs host time (pinned memory): it is made
    behind kernels that run already, and an untimed synchronous call makes no event."""
    L = Library()
    for call, kernel in ((L.attribute, "k_fix"), (L.counter, "k_counter"), (L.diff, "k_diff_join"),
                         (L.streamed, "k_fix")):
        for _ in range(20):  # (a piece of pinned memory serves several workspaces)
            L.clear()
            L.ok(call(L.ws()))
            log = L.log()
            assert first(log, kernel) < len(log)
            assert first(log, "hipHostMalloc") > first(log, kernel), log
            assert first(log, "hipEventCreate") == len(log), log


def pinned_memory_comes_in_one_piece():
    L = Library()
    n = 0
    for _ in range(16):
        L.ok(L.attribute(L.ws()))
    n = sum(x.startswith("hipHostMalloc") for x in L.log())
    assert n == 1, n


def calls_go_on_without_pinned_memory():
    """The status block is then copied after the call; the failed allocation is
    not taken for a failure of the next launch."""
    L = Library()
    for call in (L.attribute, L.counter, L.diff, L.streamed):
        L.fail("hipHostMalloc", 1000)
        L.clear()
        L.ok(call(L.ws()))
        log = L.log()
        assert first(log, "hipHostMalloc failed") < first(log, "hipMemcpyAsync .* kind 2") < len(log)
    L.fail("hipEventCreateWithFlags")
    L.ok(L.attribute(L.ws(), flags=L.N.MAG_TIME_KERNELS))  # untimed then


def kernel_attributes_do_not_change():
    """A kernel's largest LDS size is the process's: calls of any size set one value."""
    L = Library()
    for side in (5, 40, 130, 200, 600, 1100, 2500, 4096, 8192):
        L.ok(L.invariants([(side, side)]))
    values = {}
    for x in L.log():
        if x.startswith("hipFuncSetAttribute"):
            _, fn, attr, v = x.split()
            values.setdefault((fn, attr), set()).add(v)
    assert values and all(len(v) == 1 for v in values.values()), values


def _reductions(log):
    """Which reductions a call launched: groups, device-wide steps, one workgroup
    from memory; and how many times the Gram matrices were cleared."""
    return (sum(x.startswith("cooperative") for x in log), any("k_hh_reflector" in x for x in log),
            any("k_svd_eig" in x for x in log), sum("k_svd_clear" in x for x in log))


SIDES = [(600, 700), (300, 310), (130, 140)]


def groups_where_they_fit():
    L = Library()
    L.ok(L.invariants(SIDES))
    coop, steps, one, passes = _reductions(L.log())
    assert coop > 0 and not steps and not one and passes == 1


def without_groups_when_the_launch_is_refused():
    L = Library()
    for before in (0, 1):  # (1: the second launch is refused, the matrices half reduced)
        L.clear()
        L.fail("hipLaunchCooperativeKernel", 1, before)
        L.ok(L.invariants(SIDES))
        log = L.log()
        coop, steps, one, passes = _reductions(log[first(log, "CooperativeKernel failed"):])
        assert coop == 0 and steps and one and passes == 1, log
        assert _reductions(log)[3] == 2


def without_groups_when_members_lose_touch():
    L = Library()
    L.d.double_word(1)  # (the call's only 4-byte copy to the host)
    L.ok(L.invariants(SIDES))
    log = L.log()
    again = len(log) - 1 - first(log[::-1], "k_svd_clear")
    coop, steps, one, passes = _reductions(log[again:])
    assert coop == 0 and steps and one and passes == 1, log
    assert _reductions(log)[3] == 2 and _reductions(log)[0] > 0


def without_groups_on_a_masked_stream():
    L = Library()
    L.d.double_cu_mask((ctypes.c_uint32 * 8)(*[0xffffffff] * 7 + [0x7fffffff]))
    L.ok(L.invariants(SIDES))
    coop, steps, one, passes = _reductions(L.log())
    assert coop == 0 and steps and one and passes == 1


def stream_states_are_checked():
    """A state whose counts of samples, tiles and staged samples do not agree is
    refused: the next push would read its staging buffer by their difference."""
    import struct
    L = Library()
    for pushed in (0, 300, 513, 514, 5_000):
        a = L.stream(L.ws(), n=10_000)
        if pushed:
            L.ok(L.lib.mag_stream_push(a, 4096, 4096, pushed))
        n = ctypes.c_size_t(0)
        L.ok(L.lib.mag_stream_state_export(a, None, ctypes.byref(n)))
        buf = ctypes.create_string_buffer(n.value)
        L.ok(L.lib.mag_stream_state_export(a, buf, ctypes.byref(n)))
        at = 40  # magic, three sizes, streams and flags; then received, b_next, n_stage
        received, b_next, n_stage = struct.unpack_from("<3q", buf.raw, at)
        assert received == pushed and n_stage == received - 512 * b_next
        L.ok(L.lib.mag_stream_state_import(L.stream(L.ws(), n=10_000), buf, n.value))
        for bad in ((received, b_next, n_stage + 1), (received + 1, b_next, n_stage),
                    (received, b_next + 1, n_stage), (received, b_next, max(n_stage - 1, 0) + 2 * (n_stage == 0)),
                    (received, 1 << 54, n_stage)):
            bb = ctypes.create_string_buffer(buf.raw, n.value)
            struct.pack_into("<3q", bb, at, *bad)
            rc = L.lib.mag_stream_state_import(L.stream(L.ws(), n=10_000), bb, n.value)
            assert rc == L.N.MAG_E_STATE, (pushed, bad, rc)


@pytest.mark.parametrize("name", ["status_record_waits_for_the_launches",
                                  "pinned_memory_comes_in_one_piece",
                                  "calls_go_on_without_pinned_memory"])
def test_status_record(double, name):
    _run(double, name)


def test_kernel_attributes(double):
    _run(double, "kernel_attributes_do_not_change")


@pytest.mark.parametrize("name", ["groups_where_they_fit",
                                  "without_groups_when_the_launch_is_refused",
                                  "without_groups_when_members_lose_touch",
                                  "without_groups_on_a_masked_stream"])
def test_group_reductions(double, name):
    _run(double, name)


def test_stream_states(double):
    _run(double, "stream_states_are_checked")


if __name__ == "__main__":
    globals()[sys.argv[1]]()
