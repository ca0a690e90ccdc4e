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
