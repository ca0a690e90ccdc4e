"""The cooperative forms of the single-replication paths (many iterations in one launch, workgroups
exchanging tagged words) against their launch-by-launch forms, record for record. The second is
reached with a context whose memory cap leaves no room for the exchange slots, which a run
allocates last."""
import ctypes

import numpy as np
import pytest

from paper_2404_11631_amd import sim, workloads

pytestmark = pytest.mark.gpu


def both(run, records):
    """The records of `run` on an uncapped context and on one without room for the exchange."""
    out, used = [], 0
    for cap in (0, 1):
        ctx = sim.Sim(0, workspace_bytes=used - 8 if cap else 0)
        try:
            run(ctx)
            out.append(records(ctx))
            assert not cap or ctx.workspace_bytes() < used - 8      # the slots were not allocated
            used = ctx.workspace_bytes()
        finally:
            ctx.close()
    return out


def same(a, b):
    for f in a:
        assert np.array_equal(np.asarray(a[f]), np.asarray(b[f]), equal_nan=True), f


@pytest.mark.parametrize("n,S,M,R,T,x0,ckpt", [
    (4, 1, 1, 1, 1, False, ()), (4, 3, 1, 1, 40, False, (1, 2, 40)), (64, 25, 1, 1, 1030, False, (1024,)),
    (1000, 16, 3, 2, 60, True, (7,)), (260, 255, 1, 1, 30, False, ()), (4100, 33, 2, 3, 50, False, (50,)),
    (16, 50, 1, 64, 30, True, (10,)), (40_000, 12, 1, 1, 30, False, (30,)), (120_000, 50, 1, 1, 12, False, (3,))])
def test_newsvendor(n, S, M, R, T, x0, ckpt):
    print(f"[one launch] newsvendor n={n} S={S} M={M} R={R} T={T}", flush=True)
    inst = workloads.newsvendor_instance(3, 0, n)
    inst["sigma"][::7] = 0.0                        # products of certain demand: infinite thresholds
    start = 0.3 * inst["C"] / inst["c"] / n if x0 else None

    def run(ctx):
        ctx.run_newsvendor(inst, R, T, 5, S=S, M=M, x0=start, checkpoints=ckpt, gap_eps=1e3)

    def records(ctx):
        st = ctx.nv_stats()
        return dict(ctx.nv_paths(), mean=st.mean, origin=st.decision_total[0], tau_count=st.tau_count)

    a, b = both(run, records)
    same(a, b)
    assert a["cnt"].sum() == R * T


def test_exchange_slots_give_way():
    # a context that the first run fills to its cap, slots included: the second run's records need
    # the slots' room, which a context of that cap has
    inst = workloads.newsvendor_instance(3, 0, 4000)

    def two(ctx):
        for T in (40, 400):
            ctx.run_newsvendor(inst, 1, T, 5, S=16)
        return ctx.nv_paths()

    free, capped = sim.Sim(0), None
    try:
        free.run_newsvendor(inst, 1, 40, 5, S=16)
        cap = free.workspace_bytes()
        capped = sim.Sim(0, workspace_bytes=cap)
        same(two(free), two(capped))
        assert capped.workspace_bytes() <= cap
    finally:
        free.close()
        if capped:
            capped.close()


@pytest.mark.parametrize("d,N,M,R,T,w0,ckpt", [
    (4, 2, 1, 1, 1, False, ()), (128, 15, 1, 1, 40, False, (1, 40)), (132, 16, 3, 3, 1030, True, (1024,)),
    (4096, 31, 1, 1, 30, False, (30,)), (4100, 32, 2, 2, 30, True, (7,)), (8192, 63, 1, 7, 20, False, ()),
    (24_576, 8, 1, 1, 20, False, (20,)), (24_580, 25, 1, 1, 20, False, (3, 4)), (65_536, 50, 1, 1, 12, True, (12,))])
def test_wide(d, N, M, R, T, w0, ckpt):
    print(f"[one launch] wide d={d} N={N} M={M} R={R} T={T}", flush=True)
    mu, sigma = workloads.diag_instance(3, 0, d, "paper")
    p = sim.Problem(mu=mu, sigma=sigma, N=N, M=M, w0=np.full(d, 0.5 / d) if w0 else None, checkpoints=ckpt, gap_eps=0.02)

    def run(ctx):
        ctx.run_wide(p, R, T, 5)

    def records(ctx):
        st = ctx.wide_stats()
        return dict(ctx.wide_paths(), mean=st.mean, origin=st.decision_total[0], tau_count=st.tau_count)

    a, b = both(run, records)
    same(a, b)
    assert a["cnt"].sum() == R * T


@pytest.mark.parametrize("n,m,S,M,R,T,x0,ckpt", [
    (4, 1, 1, 1, 1, 1, False, ()), (8, 2, 7, 2, 3, 40, True, (1, 40)), (100, 8, 25, 1, 1, 60, False, (7,)),
    (1000, 3, 25, 1, 7, 300, False, (256,)), (3840, 3, 16, 3, 1, 30, True, ()), (3844, 3, 31, 1, 1, 30, False, (3, 4)),
    (15_360, 2, 5, 1, 1, 12, False, (12,)), (260, 5, 128, 1, 1, 20, False, ()), (332, 6, 23, 1, 1, 513, False, ())])
def test_newsvendor_constraints(n, m, S, M, R, T, x0, ckpt):
    print(f"[one launch] constraints n={n} rows={m} S={S} M={M} R={R} T={T}", flush=True)
    inst = workloads.newsvendor_instance(3, 0, n)
    inst["sigma"][::7] = 0.0
    A, C = workloads.newsvendor_constraints(3, 0, n, m)
    start = np.full(n, 0.25 * float(np.min(C / A.sum(axis=1)))) if x0 else None

    def run(ctx):
        ctx.run_newsvendor_lp(inst, A, C, R, T, 5, S=S, M=M, x0=start, checkpoints=ckpt, gap_eps=1e3)

    def records(ctx):
        st = ctx.nv_lp_stats()
        return dict(ctx.nv_lp_paths(), mean=st.mean, origin=st.decision_total[0], tau_count=st.tau_count)

    a, b = both(run, records)
    same(a, b)
    assert a["pivots"].max() <= sim.NV_LP_MAX_PIVOTS


@pytest.mark.parametrize("n,rows,b,bH,M,L,R,K,fp32,ckpt", [
    (1, 64, 1, 1, 1, 1, 1, 1, False, ()), (50, 400, 20, 30, 4, 3, 7, 40, False, (7, 22)), (256, 300, 64, 64, 5, 2, 1, 30, True, ()),
    (260, 500, 65, 24, 32, 1, 2, 60, False, (5,)), (1000, 700, 300, 600, 25, 10, 1, 60, False, (41,)),
    (5000, 900, 50, 300, 25, 10, 3, 300, False, (20, 300)), (8192, 600, 50, 301, 2, 3, 1, 20, False, ()),
    (300, 500, 10, 12, 3, 2, 1, 4100, False, (4096, 4097))])
def test_sqn_split(n, rows, b, bH, M, L, R, K, fp32, ckpt):
    print(f"[one launch] sqn n={n} b={b} bH={bH} M={M} L={L} R={R} K={K} fp32={fp32}", flush=True)
    rng = np.random.default_rng(3)
    X = (rng.random((rows, n)) < min(0.5, 25.0 / n)).astype(np.uint8)
    z = rng.integers(0, 2, rows).astype(np.uint8)

    def run(ctx):
        ctx.sqn_load(X, z)
        ctx.run_sqn(R, K, 5, L=L, M=M, b=b, bH=bH, checkpoints=ckpt, pairs_fp32=fp32, split=True)

    def records(ctx):
        st = ctx.sqn_stats()
        return dict(ctx.sqn_paths(), mean=st.mean)

    a, b2 = both(run, records)
    same(a, b2)
    assert a["pairs"].tolist() == [max(K // L - 1, 0)] * R


def test_sqn_split_captured():
    # a captured run is replayed with eager runs in between: every replay leaves the eager run's iterates
    rng = np.random.default_rng(6)
    X, z = (rng.random((400, 300)) < 0.1).astype(np.uint8), rng.integers(0, 2, 400).astype(np.uint8)
    ctx, vp = sim.Sim(0), ctypes.c_void_p
    stream, graph, replay = vp(), vp(), vp()

    def hip(name, *args):                     # the runtime that the library is linked with
        assert getattr(ctx.L, name)(*args) == 0, name

    def run(seed):
        ctx.run_sqn(2, 40, seed, L=4, M=5, b=20, bH=40, checkpoints=(), split=True)

    try:
        hip("hipStreamCreate", ctypes.byref(stream))
        ctx.set_stream(stream.value)
        ctx.sqn_load(X, z)
        run(6)
        want, view = ctx.sqn_paths()["w"], sim.SimSqnView()
        ctx._check(ctx.L.sim_sqn_paths(ctx.h, ctypes.byref(view)))
        hip("hipStreamBeginCapture", stream, 1)
        run(6)
        hip("hipStreamEndCapture", stream, ctypes.byref(graph))
        hip("hipGraphInstantiate", ctypes.byref(replay), graph, None, None, ctypes.c_size_t(0))
        for k in range(3):
            print(f"[one launch] sqn graph replay {k}", flush=True)
            run(7 + k)
            assert not np.array_equal(ctx.sqn_paths()["w"], want)
            hip("hipGraphLaunch", replay, stream)
            hip("hipStreamSynchronize", stream)
            w = ctx._copy(view.w, np.float64, 2 * view.ld).reshape(2, view.ld)[:, :300]
            assert np.array_equal(w, want)
        hip("hipGraphExecDestroy", replay)
        hip("hipGraphDestroy", graph)
    finally:
        ctx.close()


def compare_split(d, N, M, R, T, ckpt, features=False, precision=sim.FP32):
    print(f"[one launch] paths d={d} N={N} M={M} R={R} T={T} features={features} precision={precision}", flush=True)
    mu, sigma = workloads.diag_instance(15, d, d)
    p = sim.Problem(mu=mu, sigma=sigma, N=N, M=M, checkpoints=ckpt, gap_eps=0.05, cv_features=features,
                    cv_ref=-mu if features else None, w0=np.full(d, 0.5 / d) if R == 300 else None, instance_id=d,
                    log_reps=(0, min(R, 8)), precision=precision)

    def run(ctx):
        ctx.run(p, R, T, 5)

    def records(ctx):
        st, g = ctx.stats(), ctx.paths()
        out = {f: getattr(st, f) for f in ("mean", "var", "min", "max", "tau_count", "tau_mean")}
        out.update(total=list(st.decision_total), sd=list(st.f_sd)[:len(ckpt)], rse=list(st.rse_mean)[:len(ckpt)],
                   decisions=g["decisions"], f=g.get("f_ckpt", 0))
        if features:
            out["x"] = g["x"]
        return out

    a, b = both(run, records)
    same(a, b)


@pytest.mark.parametrize("d,N,M,R,T,ckpt,features", [
    (2, 2, 1, 1, 1, (), False), (3, 5, 1, 64, 40, (1, 40), False), (4, 9, 3, 65, 37, (7,), False), (5, 3, 1, 300, 25, (), True),
    (7, 6, 1, 257, 30, (30,), False), (10, 11, 2, 130, 33, (2, 33), False), (10, 10, 1, 100, 200, (), True), (13, 2, 1, 70, 40, (), False),
    (15, 7, 1, 64, 30, (3,), False), (17, 5, 2, 100, 31, (), False), (21, 6, 1, 90, 20, (), True), (27, 31, 1, 65, 20, (20,), False),
    (30, 3, 1, 63, 20, (), False), (31, 8, 1, 129, 20, (), False), (32, 4, 1, 300, 20, (5,), False), (12, 3, 1, 49_000, 12, (), False)])
def test_paths_drawn_by_other_wavefronts(d, N, M, R, T, ckpt, features):
    # against a lane per replication, which a context without room for the records takes: odd groups, halves
    # of long groups, partial units, chunks across iterations, features
    compare_split(d, N, M, R, T, ckpt, features)


@pytest.mark.parametrize("d,N,M,R,T,ckpt", [
    (1, 2, 1, 1, 1, ()), (1, 9, 2, 65, 37, (3, 37)), (2, 2, 1, 1000, 100, (100,)), (5, 7, 1, 64, 30, ()), (7, 6, 3, 300, 25, (25,)),
    (9, 5, 1, 130, 20, ()), (10, 3, 1, 63, 40, (1,)), (13, 4, 1, 100, 20, ()), (15, 7, 2, 70, 20, (20,)), (16, 5, 1, 129, 20, ())])
def test_binary64_paths_drawn_by_other_wavefronts(d, N, M, R, T, ckpt):
    compare_split(d, N, M, R, T, ckpt, precision=sim.FP64)


@pytest.mark.parametrize("n,M,b,bH,R", [(1, 1, 1, 1, 2), (60, 32, 1024, 300, 3), (1000, 25, 50, 300, 300), (1024, 4, 33, 1024, 2),
                                        (1028, 4, 9, 20, 257), (2048, 3, 5, 7, 260), (2600, 25, 50, 90, 2), (4100, 2, 40, 65, 2)])
def test_sqn_replications_do_not_depend_on_their_number(n, M, b, bH, R):
    # the threads of a workgroup and the rows staged at a time follow from the sizes and from R: a
    # replication alone and among R others is the same bits
    print(f"[one launch] sqn n={n} M={M} b={b} bH={bH} R={R}", flush=True)
    rng = np.random.default_rng(4)
    X = (rng.random((500, n)) < min(0.5, 25.0 / n)).astype(np.uint8)
    z = rng.integers(0, 2, 500).astype(np.uint8)
    ctx = sim.Sim(0)
    try:
        ctx.sqn_load(X, z)
        ctx.run_sqn(R, 30, 5, L=3, M=M, b=b, bH=bH, checkpoints=(7, 30))
        a, st = ctx.sqn_paths(), ctx.sqn_stats()
        ctx.run_sqn(1, 30, 5, L=3, M=M, b=b, bH=bH, checkpoints=(7, 30))
        c = ctx.sqn_paths()
    finally:
        ctx.close()
    for f in ("w", "S", "Y", "pairs"):
        assert np.array_equal(np.asarray(a[f][0]), np.asarray(c[f][0]), equal_nan=True), f
    assert np.array_equal(a["w_ckpt"][:, 0], c["w_ckpt"][:, 0], equal_nan=True)
    if np.isfinite(a["F"]).all():           # a pair without curvature (one feature, one row) divides by 0
        assert st.min == a["F"].min() and st.max == a["F"].max()
        assert st.f_mean[0] == pytest.approx(a["F_ckpt"][0].mean(), rel=1e-13)
