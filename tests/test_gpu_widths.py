"""The exact-width path kernels (one per asset count up to 32) at the edges of their sample groups:
N below, at and past a whole group of Philox blocks, against the oracle by the protocol of parity.py,
and the feature-writing kernel of the same width against the plain one, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2404_11631_amd import sim, workloads
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    s = sim.Sim(0)
    yield s
    s.close()


def check(ctx, p, R, T, seed):
    print(f"[widths] d={len(p.mu)} N={p.N} noise={p.noise} R={R} T={T}", flush=True)
    ctx.run(p, R, T, seed)
    st, g = ctx.stats(), ctx.paths()
    P = parity.oracle_problem(p, seed)
    outs = (oracle.PathOut * R)()
    for r in range(R):
        outs[r] = parity.check_rep(P, g, r, T, parity.uroff(p), decisions=g["decisions"][:, r])
    parity.check_stats(st, P.reduce(outs, T), len(p.checkpoints), len(p.mu), g["tau"])
    return g


@pytest.mark.parametrize("d,N,noise", [
    (7, 3, sim.NOISE_GAUSS), (7, 6, sim.NOISE_GAUSS), (9, 9, sim.NOISE_GAUSS), (11, 2, sim.NOISE_GAUSS),
    (1, 23, sim.NOISE_GAUSS), (2, 13, sim.NOISE_GAUSS), (4, 7, sim.NOISE_GAUSS), (14, 5, sim.NOISE_GAUSS),
    (17, 6, sim.NOISE_GAUSS), (23, 7, sim.NOISE_GAUSS), (26, 5, sim.NOISE_GAUSS), (27, 31, sim.NOISE_GAUSS),
    (31, 3, sim.NOISE_GAUSS), (1, 11, sim.NOISE_T), (5, 6, sim.NOISE_T), (13, 7, sim.NOISE_T), (20, 3, sim.NOISE_T),
    (29, 5, sim.NOISE_T), (32, 4, sim.NOISE_T)])
def test_width(ctx, d, N, noise):
    mu, sigma = workloads.diag_instance(11, d, d)
    p = sim.Problem(mu=mu, sigma=sigma, N=N, M=1 + d % 2, noise=noise, nu=3, checkpoints=(5, 40), gap_eps=0.05,
                    instance_id=d, keep_paths=True, log_reps=(0, 70))
    check(ctx, p, 70, 40, seed=77 + d)


@pytest.mark.parametrize("d,N", [(7, 6), (10, 10), (13, 5), (27, 7)])
def test_features_same_paths(ctx, d, N):
    mu, sigma = workloads.diag_instance(12, d, d)
    kw = dict(mu=mu, sigma=sigma, N=N, checkpoints=(30,), keep_paths=True)
    ctx.run(sim.Problem(**kw), 300, 60, 5)
    a = ctx.paths()
    ctx.run(sim.Problem(cv_features=True, cv_ref=-mu, **kw), 300, 60, 5)
    b = ctx.paths()
    for f in ("y", "f_ckpt", "cnt", "wsum", "tau"):
        assert np.array_equal(a[f], b[f]), f


@pytest.mark.parametrize("split,N,noise", [(1, 5, sim.NOISE_GAUSS), (1, 9, sim.NOISE_T), (2, 6, sim.NOISE_GAUSS), (4, 13, sim.NOISE_GAUSS),
                                           (8, 3, sim.NOISE_GAUSS), (8, 40, sim.NOISE_T), (16, 33, sim.NOISE_GAUSS)])
def test_tile_widths(ctx, split, N, noise):
    # every width at `split` sample lanes: last rounds shorter than the others, an odd number of blocks,
    # chunks without samples
    probs, P = [], []
    for d in range(1, 33):
        mu, sigma = workloads.diag_instance(13, d, d)
        probs.append(sim.Problem(mu=mu, sigma=sigma, N=N, M=1 + d % 2, noise=noise, nu=3, checkpoints=(5, 70), gap_eps=0.05,
                                 instance_id=d, log_reps=(0, 3)))
        P.append(min(64, split * (1 if d <= 8 else 2 if d <= 16 else 4)))
    print(f"[widths] tiles split={split} N={N} noise={noise}", flush=True)
    ctx.run_batch(probs, [3] * 32, [70] * 32, 9, lanes_per_rep=P, keep_paths=True)
    for i, p in enumerate(probs):
        st, g = ctx.batch_stats(i), ctx.batch_paths(i)
        op = parity.oracle_problem(p, 9)
        for r in range(3):
            parity.check_rep(op, g, r, 70, oracle.U32, decisions=g["decisions"][:, r])
        assert list(st.decision_total)[:len(p.mu) + 1] == g["cnt"].sum(axis=1).tolist()
        assert st.mean == pytest.approx(g["y"].mean(), rel=1e-12) and st.R == 3


@pytest.mark.parametrize("d,N,M", [(1, 2, 1), (16, 16, 1), (16, 17, 2), (17, 16, 1), (3, 32, 1), (32, 32, 3), (32, 33, 1), (8, 32, 1),
                                   (9, 29, 1), (5, 100, 2), (4, 527, 1)])
def test_one_replication_per_wavefront(ctx, d, N, M):
    # the edges of the register forms, one and three drawing wavefronts, epochs of several iterations
    mu, sigma = workloads.diag_instance(14, d, d)
    p = sim.Problem(mu=mu, sigma=sigma, N=N, M=M, checkpoints=(5, 70), gap_eps=0.05, w0=np.full(d, 0.5 / d), instance_id=d,
                    log_reps=(0, 3))
    print(f"[widths] wavefront d={d} N={N} M={M}", flush=True)
    ctx.run_batch([p], [3], [70], 9, lanes_per_rep=[64], keep_paths=True)
    st, g = ctx.batch_stats(0), ctx.batch_paths(0)
    op = parity.oracle_problem(p, 9)
    for r in range(3):
        parity.check_rep(op, g, r, 70, oracle.U32, decisions=g["decisions"][:, r])
    assert list(st.decision_total)[:d + 1] == g["cnt"].sum(axis=1).tolist()


@pytest.mark.parametrize("d,N,R,T,features,mean", [
    (1, 7, 8192, 3000, False, "0x1.5aa84d8c3f40ep-6"), (2, 3, 60_000, 1500, False, "-0x1.3579d6ece3074p-1"),
    (2, 3, 60_000, 1500, True, "-0x1.3579d6ece3074p-1"), (10, 5, 8192, 3000, False, "-0x1.cca8b498cd351p-1"),
    (10, 5, 8192, 3000, True, "-0x1.cca8b498cd351p-1"), (10, 5, 60_000, 1500, False, "-0x1.cca5956864ad8p-1"),
    (2, 5, 1000, 93_000, False, "-0x1.46fc73d6f19b0p-1"), (10, 3, 1000, 93_000, False, "-0x1.c9ed2be147d08p-1")])
def test_partial_group_decisions(ctx, d, N, R, T, features, mean):
    # N past a whole group of Philox blocks, at the widths whose last samples fuse into s1 as the others do:
    # one rounding more there decides a near tie in ~1e7 iterations the other way, which shows in the mean of
    # Y. The values are those of the kernels before there was one for every width.
    print(f"[widths] partial group d={d} N={N} R={R} T={T} features={features}", flush=True)
    mu, sigma = workloads.diag_instance(1, 0, d)
    ctx.run(sim.Problem(mu=mu, sigma=sigma, N=N, checkpoints=(T,), cv_features=features, cv_ref=-mu if features else None), R, T, 5)
    assert ctx.stats().mean.hex() == mean


@pytest.mark.parametrize("d,limit,precision", [(2, 32_768, sim.FP32), (3, 49_152, sim.FP32), (10, 49_152, sim.FP32),
                                               (3, 32_768, sim.FP64), (4, 49_152, sim.FP64), (10, 32_768, sim.FP64)])
def test_split_form_ends(d, limit, precision):
    # the split form leaves records, which a run that keeps none has a buffer for: up to `limit` replications,
    # so the tests past it reach the kernels of one lane per replication
    mu, sigma = workloads.diag_instance(16, d, d)
    used = []
    for R in (limit, limit + 1):
        print(f"[widths] form d={d} R={R} precision={precision}", flush=True)
        s = sim.Sim(0)
        try:
            s.run(sim.Problem(mu=mu, sigma=sigma, N=5, precision=precision), R, 2, 1)
            used.append(s.workspace_bytes())
        finally:
            s.close()
    assert used[0] - used[1] > limit * (8 + 4 * (d + 2)) - 65_536


@pytest.mark.parametrize("features", [False, True])
@pytest.mark.parametrize("d,N,M", [(1, 6, 1), (2, 5, 2), (6, 3, 1), (7, 6, 2), (10, 5, 1), (13, 7, 1), (16, 3, 2), (27, 7, 1), (31, 3, 1),
                                   (32, 5, 2)])
def test_one_lane_per_replication(ctx, d, N, M, features):
    # past the split form: the last replications (the last alone in its workgroup) against the oracle, and
    # the records of all against the statistics
    R, T = 49_153, 24
    print(f"[widths] one lane d={d} N={N} M={M} features={features}", flush=True)
    mu, sigma = workloads.diag_instance(16, d, d)
    p = sim.Problem(mu=mu, sigma=sigma, N=N, M=M, checkpoints=(5, T), gap_eps=0.05, w0=np.full(d, 0.5 / d), instance_id=d,
                    keep_paths=True, log_reps=(R - 4, 4), cv_features=features, cv_ref=-mu if features else None)
    ctx.run(p, R, T, 21 + d)
    st, g = ctx.stats(), ctx.paths()
    P = parity.oracle_problem(p, 21 + d)
    for r in range(R - 4, R):
        parity.check_rep(P, g, r, T, oracle.U32, decisions=g["decisions"][:, r - (R - 4)])
    assert (g["cnt"].sum(axis=0) == T).all()
    assert list(st.decision_total)[:d + 1] == g["cnt"].sum(axis=1, dtype=np.uint64).tolist()
    hit = g["tau"] != oracle.TAU_NONE
    assert st.tau_count == hit.sum() and st.min == g["y"].min() and st.max == g["y"].max()
    # a plain sum of R values is within R roundings of the exact one
    assert st.mean == pytest.approx(g["y"].mean(), rel=R * 2.0 ** -53)


@pytest.mark.parametrize("d,N", [(2, 5), (7, 6), (10, 10), (13, 5), (27, 7), (32, 3)])
def test_one_lane_features_same_paths(ctx, d, N):
    mu, sigma = workloads.diag_instance(12, d, d)
    kw = dict(mu=mu, sigma=sigma, N=N, checkpoints=(30,), keep_paths=True)
    ctx.run(sim.Problem(**kw), 49_153, 30, 5)
    a = ctx.paths()
    ctx.run(sim.Problem(cv_features=True, cv_ref=-mu, **kw), 49_153, 30, 5)
    b = ctx.paths()
    for f in ("y", "f_ckpt", "cnt", "wsum", "tau"):
        assert np.array_equal(a[f], b[f]), f
