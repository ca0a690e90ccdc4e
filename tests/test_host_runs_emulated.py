"""The host side of the runs that take one cooperative launch (wide, newsvendor, constraints, split SQN) with
their real kernels on a CPU runtime (tests/emu/emu_runtime.hpp): the library's own sources, a process
per workgroup of a cooperative launch. The cooperative form against the launch-by-launch form, bit for
bit, and what happens when it goes wrong: a wait that gives up, before a launch or within it."""
import ctypes
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_2404_11631_amd import sim, workloads

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = ("wide_api.hip", "nv_api.hip", "sqn_api.hip", "sim_api.hip", "fw_wide.hip", "fw_wide_run.hip", "fw_newsvendor.hip",
           "fw_newsvendor_run.hip", "fw_newsvendor_lp_run.hip", "fw_sqn_split.hip", "fw_sqn_split_run.hip", "host_core.cpp")
WIDE, NEWSVENDOR, CONSTRAINTS, SQN = KINDS = (1, 2, 3, 4)


class Faults(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("refuse", "missing", "failed", "fail_launch", "none", "cooperative", "launches")]


class Lib:
    """The emulated library; sim.load() also names the entry points that it leaves out."""

    def __init__(self, path):
        self.real = ctypes.CDLL(path)
        self.real.emu_faults.restype = ctypes.POINTER(Faults)
        self.real.emu_log.restype = ctypes.c_char_p

    def __getattr__(self, name):
        try:
            return getattr(self.real, name)
        except AttributeError:
            if not name.startswith("sim_"):
                raise
            return type("LeftOut", (), {})()


@pytest.fixture(scope="module")
def build(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("host_emu")
    flags = ["-std=c++20", "-O2", "-fPIC", "-w", "-I", os.path.join(HERE, "emu", "shim"), "-I", os.path.join(ROOT, "include"),
             "-I", os.path.join(HERE, "emu")]

    def compile_one(limit, src, obj):
        hip = src.endswith(".hip")
        cmd = [gxx, *flags, f"-DFW_POLL_LIMIT={limit}", *(["-include", "emu_runtime.hpp", "-x", "c++"] if hip else []), "-c", src, "-o", obj]
        subprocess.check_call(cmd)
        return obj

    def make(limit):
        so = str(d / f"libemu{limit}.so")
        if not os.path.exists(so):
            srcs = [os.path.join(ROOT, "paper_2404_11631_amd", "csrc", s) for s in SOURCES] + [os.path.join(HERE, "emu", "emu_host.cpp")]
            with ThreadPoolExecutor(8) as ex:
                objs = list(ex.map(lambda s: compile_one(limit, s, str(d / f"{limit}_{os.path.basename(s)}.o")), srcs))
            subprocess.check_call([gxx, "-shared", "-o", so, *objs, "-lpthread"])
        return so
    return make


@pytest.fixture
def emu(build, monkeypatch):
    """emu(limit): the emulated library with that poll limit, in place of the built one."""
    def load(limit=1 << 20):
        lib = Lib(build(limit))
        with monkeypatch.context() as m:
            m.setattr(sim, "_lib", None)
            m.setattr(sim, "LIB_PATH", lib.real._name)
            m.setattr(sim.ctypes, "CDLL", lambda path: lib)
            loaded = sim.load()
        monkeypatch.setattr(sim, "_lib", loaded)
        return lib
    return load


def set_faults(lib, kind, **faults):
    lib.emu_reset()
    lib.emu_kind(kind)
    for k, v in faults.items():
        setattr(lib.emu_faults()[0], k, v)


# two or three cooperative launches each: a checkpoint ends one (the SQN run has one launch of 4,096 steps)
def start(kind, ctx, R=1, big=False):
    if kind == WIDE:
        mu, sigma = workloads.diag_instance(3, 0, 388 if big else 260, "paper")
        p = sim.Problem(mu=mu, sigma=sigma, N=5, M=2, checkpoints=(1, 2), gap_eps=0.02, w0=np.full(len(mu), 0.5 / len(mu)))
        ctx.run_wide(p, R, 3, 5)
    elif kind == NEWSVENDOR:
        inst = workloads.newsvendor_instance(3, 0, 516 if big else 260)
        inst["sigma"][::7] = 0.0
        ctx.run_newsvendor(inst, R, 3, 5, S=5, M=2, checkpoints=(1, 2), gap_eps=1e3, x0=0.3 * inst["C"] / inst["c"] / len(inst["c"]))
    elif kind == CONSTRAINTS:
        n = 200 if big else 100
        inst = workloads.newsvendor_instance(3, 0, n)
        inst["sigma"][::7] = 0.0
        A, C = workloads.newsvendor_constraints(3, 0, n, 2)
        x0 = np.full(n, 0.25 * float(np.min(C / A.sum(axis=1))))
        ctx.run_newsvendor_lp(inst, A, C, R, 3, 5, S=5, M=2, checkpoints=(1, 2), gap_eps=1e3, x0=x0)
    else:
        rng = np.random.default_rng(3)
        n = 520 if big else 300
        ctx.sqn_load((rng.random((60, n)) < 0.1).astype(np.uint8), rng.integers(0, 2, 60).astype(np.uint8))
        ctx.run_sqn(R, 12, 5, L=2, M=3, b=20 if big else 5, bH=7, checkpoints=(3, 8), split=True)


def stats(kind, ctx):
    return (None, ctx.wide_stats, ctx.nv_stats, ctx.nv_lp_stats, ctx.sqn_stats)[kind]()


def paths(kind, ctx):
    return (None, ctx.wide_paths, ctx.nv_paths, ctx.nv_lp_paths, ctx.sqn_paths)[kind]()


def records(kind, ctx, paths_first=False):
    g = paths(kind, ctx) if paths_first else None
    st = stats(kind, ctx)
    return dict(g or paths(kind, ctx), mean=st.mean, var=st.var, min=st.min, max=st.max, origin=st.decision_total[0], tau_count=st.tau_count,
                f_mean=list(st.f_mean)[:2])


def run(lib, kind, R=1, paths_first=False, **faults):
    set_faults(lib, kind, **faults)
    ctx = sim.Sim(0)
    try:
        start(kind, ctx, R)
        out = records(kind, ctx, paths_first)
    finally:
        ctx.close()
    return out, lib.emu_faults()[0].cooperative, lib.emu_faults()[0].launches


by_launches = {}


def wanted(lib, kind, R=1):
    """The records and the launches of the launch-by-launch form."""
    if (kind, R) not in by_launches:
        out, cooperative, launches = run(lib, kind, R, none=1)
        assert cooperative == 0
        by_launches[kind, R] = out, launches
    return by_launches[kind, R]


def same(a, b):
    assert a.keys() == b.keys()
    for f in a:
        assert np.array_equal(np.asarray(a[f]), np.asarray(b[f]), equal_nan=True), f


@pytest.mark.parametrize("kind", KINDS)
def test_same_bits(emu, kind):
    lib = emu()
    want, by_launch = wanted(lib, kind, 2)
    got, cooperative, launches = run(lib, kind, 2)
    same(got, want)
    assert cooperative == (1 if kind == SQN else 3) and launches < by_launch


LAUNCHES = [(k, f) for k in KINDS for f in ((0,) if k == SQN else (0, 1, 2))]


@pytest.mark.parametrize("kind,failed", LAUNCHES)
def test_wait_gave_up_before_a_launch(emu, kind, failed):
    # the failure word is up when launch `failed` starts, the ones before it have run: the repeat starts over,
    # whichever of the results is read first
    lib = emu()
    want, by_launch = wanted(lib, kind)
    got, _, launches = run(lib, kind, paths_first=failed != 1, failed=failed)
    same(got, want)
    assert launches > by_launch


@pytest.mark.parametrize("kind,missing", LAUNCHES)
def test_wait_gives_up_in_a_launch(emu, kind, missing):
    # a workgroup is missing in a launch: every wait for it ends, the others leave, and the run is repeated
    # (with 64 polls a wait may also give up by itself)
    lib = emu(64)
    want, by_launch = wanted(lib, kind)
    got, cooperative, launches = run(lib, kind, missing=missing)
    same(got, want)
    assert cooperative and launches > by_launch


@pytest.mark.parametrize("at", [0, 2])
@pytest.mark.parametrize("kind", KINDS)
def test_repeat_fails(emu, kind, at):
    # the repeat of a run that gave up fails (its ordinary launch `at`): no result of the abandoned run is
    # handed out, then or later, and once launches work again the results are right or still an error
    lib = emu()
    want, _ = wanted(lib, kind)
    set_faults(lib, kind, failed=0)
    ctx = sim.Sim(0)
    try:
        start(kind, ctx)
        lib.emu_faults()[0].fail_launch = lib.emu_faults()[0].launches + at
        for read in (stats, paths, stats):
            with pytest.raises(sim.SimError):
                read(kind, ctx)
        lib.emu_faults()[0].fail_launch = -1
        same(records(kind, ctx), want)
    finally:
        ctx.close()


@pytest.mark.parametrize("kind,refuse", LAUNCHES)
def test_launch_refused(emu, kind, refuse):
    # a cooperative launch that the runtime refuses, the first or a later one: the launch-by-launch form
    lib = emu()
    want, by_launch = wanted(lib, kind)
    got, cooperative, launches = run(lib, kind, refuse=refuse)
    same(got, want)
    assert cooperative == refuse + 1 and launches >= by_launch


@pytest.mark.parametrize("kind", [CONSTRAINTS, SQN])
def test_function_attribute_does_not_follow_the_run(emu, kind):
    # the LDS that a kernel may take is set for the function, which every context and thread shares: a smaller
    # run must not lower it between a larger one's check and its launch
    lib = emu()
    set_faults(lib, kind, refuse=0)
    ctx = sim.Sim(0)
    try:
        for big in (True, False):
            if kind == CONSTRAINTS:
                n = 5120 if big else 4096
                A, C = workloads.newsvendor_constraints(3, 0, n, 2)
                ctx.run_newsvendor_lp(workloads.newsvendor_instance(3, 0, n), A, C, 1, 1, 5, S=2)
            else:
                start(SQN, ctx, big=big)
            lib.emu_faults()[0].refuse = 1
    finally:
        ctx.close()
    values = {}
    for line in lib.emu_log().decode().split("\n"):
        if line.startswith("attribute"):
            _, fn, value = line.split()
            values.setdefault(fn, []).append(value)
    assert values
    for fn, v in values.items():
        assert len(set(v)) == 1, v


@pytest.mark.parametrize("kind", [0, *KINDS])
def test_timed_interval_holds_no_allocation(emu, kind):
    # a first run's device time (between two events) does not include the allocation of its scratch
    lib = emu()
    set_faults(lib, kind)
    ctx = sim.Sim(0)
    try:
        if kind:
            start(kind, ctx)
        else:
            ctx.run(sim.Problem(mu=np.ones(3), sigma=np.ones(3), N=5), 100, 5, 1)
    finally:
        log = lib.emu_log().decode().split("\n")
        ctx.close()
    events = [i for i, line in enumerate(log) if line == "event"]
    assert len(events) >= 2 and "malloc" in log[:events[0]]
    assert not {"malloc", "free"} & set(log[events[0]:events[-1]])
