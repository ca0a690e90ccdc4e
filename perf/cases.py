"""Workloads whose run time this repository looks after, through the public binding in ``sim.py``.

Every case is what a program that uses the framework calls: a simulation and the statistics (and,
where kept, the records) it leaves. Sizes are the repository's named workloads and Section 4.1's
experiments, with reduced replication counts where a full run takes longer than two seconds.

    listed()            the cases, dicts of plain values
    draw(rng)           one more case of the same ranges
    prepare(case, seed) a context and the inputs of one call, made from the seed
    run(state)          one call and its outputs
    work(case)          bytes and operations the method cannot do without
    exact(case, seed)   the floating outputs in 64 bits, by plain torch and numpy

Operations are counted as in the benchmark: 23 per standard normal (generator, uniform map,
Box-Muller, the one-pass statistics), 25 per demand sample, 15 per asset and iteration.
"""
import math

import numpy as np
import torch

from paper_2404_11631_amd import sim, workloads

TABLE2 = (50, 100, 500, 1000)
EXACT_NORMALS = 2e10            # beyond this many normals exact() would take too long
CHUNK = 1 << 24                 # normals held at once by exact()


def _ckpt(T):
    return tuple(c for c in TABLE2 if c < T) + (T,)


def listed():
    return [
        # the tiny workload: one small FP64 study with its per-path records; a call's latency
        dict(name="paths_tiny_fp64", kind="paths", R=1000, T=100, d=2, N=2, M=1, fp64=True, t_noise=False, keep=True),
        # the benchmark's paper-scale workload: a million replications, ten assets
        dict(name="paths_paper_scale", kind="paths", R=1_000_000, T=10_000, d=10, N=10, M=1, fp64=False, t_noise=False,
             keep=False),
        # a study at a width that is no power of two, with records
        dict(name="paths_ragged_d27", kind="paths", R=65_000, T=400, d=27, N=31, M=1, fp64=False, t_noise=False, keep=True),
        # the stress workload's instance (dense factor, heavy tails), fewer replications and steps
        dict(name="dense_stress", kind="dense", R=100_000, T=200, d=64, N=100, t_noise=True),
        # a batch of instances of uneven size and horizon
        dict(name="batch_uneven", kind="batch", n_inst=64, R=1024, t_hi=10_000, lanes=0, shape=0),
        # the shortest confidence interval: 1,024 paths of the paper-scale instance, latency-bound
        dict(name="batch_latency", kind="latency", R=1024, T=10_000, d=10, N=10),
        # the control variate: train on simulated pairs, then one estimate
        dict(name="control_variate", kind="cv", R_train=65_536, R=65_536, T=500, d=10, N=10, epochs=2, batch=4096),
        # Section 4.1's Task 1: one replication, many assets
        dict(name="wide_10k", kind="wide", R=1, T=1500, d=10_000, N=25, M=1),
        # Section 4.1's Task 2: the newsvendor, one resource row
        dict(name="newsvendor_10k", kind="newsvendor", R=1, T=1500, n=10_000, S=25, M=1),
        # Task 2 over a general technology matrix
        dict(name="newsvendor_lp_1k", kind="lp", R=1, T=1500, n=1000, S=25, resources=3, M=1),
        # Section 4.1's Task 3: one run of the largest data set
        dict(name="sqn_single_5k", kind="sqn", R=1, K=2000, n=5000, rows=150_000, b=50, bH=300, split=True, fp32=False),
        # Task 3 over many replications of the mid-sized data set (confidence intervals of its loss)
        dict(name="sqn_batch_1k", kind="sqn", R=512, K=500, n=1000, rows=30_000, b=50, bH=300, split=False, fp32=False),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["paths", "paths", "paths", "dense", "batch", "latency", "wide", "wide", "newsvendor", "newsvendor",
                       "lp", "sqn", "sqn", "cv"])
    if kind == "paths":
        fp64, t_noise = rng.random() < 0.2, rng.random() < 0.2
        d, N = rng.randint(1, 16 if fp64 else 32), _log(rng, 2, 60)
        T, M = _log(rng, 100, 10_000), rng.choice([1, 1, 1, 2, 5])
        cap = 4e9 if fp64 else 2e10
        R = max(64, min(_log(rng, 500, 1_000_000), int(cap / (T * N * d))))
        return dict(kind=kind, R=R, T=T, d=d, N=N, M=M, fp64=fp64, t_noise=t_noise, keep=rng.random() < 0.4)
    if kind == "dense":
        d, N, T = rng.choice([32, 64]), rng.randint(10, 100), _log(rng, 50, 1000)
        R = max(64, min(_log(rng, 2000, 200_000), int(2e10 / (T * N * d))))
        return dict(kind=kind, R=R, T=T, d=d, N=N, t_noise=rng.random() < 0.6)
    if kind == "batch":
        return dict(kind=kind, n_inst=rng.randint(8, 128), R=_log(rng, 100, 1500), t_hi=_log(rng, 1000, 10_000), lanes=0,
                    shape=rng.randint(1, 1 << 20))
    if kind == "latency":
        d = rng.randint(2, 32)
        return dict(kind=kind, R=_log(rng, 50, 2000), T=_log(rng, 500, 10_000), d=d, N=rng.randint(2, 2100 // d // 2))
    if kind == "cv":
        b = 128 * rng.randint(4, 64)
        return dict(kind=kind, R_train=b * rng.randint(4, 16), R=_log(rng, 5000, 100_000), T=_log(rng, 100, 1000),
                    d=rng.randint(2, 16), N=rng.randint(2, 20), epochs=rng.randint(1, 3), batch=b)
    if kind == "wide":
        d = 4 * _log(rng, 25, 25_000)
        return dict(kind=kind, R=rng.choice([1, 1, 7]), T=_log(rng, 300, 1500), d=d, N=rng.randint(10, 50),
                    M=rng.choice([1, 1, 3]))
    if kind == "newsvendor":
        n = 4 * _log(rng, 25, 250_000)
        return dict(kind=kind, R=rng.choice([1, 1, 7]) if n < 100_000 else 1, T=_log(rng, 300, 1500), n=n,
                    S=rng.randint(10, 50), M=rng.choice([1, 1, 3]))
    if kind == "lp":
        return dict(kind=kind, R=rng.choice([1, 1, 7]), T=_log(rng, 200, 1500), n=4 * _log(rng, 25, 2500),
                    S=rng.randint(10, 50), resources=rng.randint(1, 6), M=rng.choice([1, 1, 3]))
    split, n = rng.random() < 0.6, _log(rng, 50, 5000)
    return dict(kind="sqn", R=rng.choice([1, 1, 7]) if split else _log(rng, 16, 512), K=_log(rng, 200, 2000 if split else 400),
                n=n, rows=min(30 * n, 60_000), b=rng.choice([25, 50, 50, 100]), bH=rng.choice([300, 600]), split=split,
                fp32=False)


# ---- inputs -----------------------------------------------------------------------------------
def _instance(case, seed, d, i=0):
    return workloads.diag_instance(seed, i, d, "paper" if case["kind"] == "wide" else "unit")


def _sizes(case):
    """(d, N, T) of every instance of a batch; they belong to the case, the parameters to the seed."""
    return [(b.d, b.N, b.T) for b in
            workloads.uneven_batch(case["shape"], case["n_inst"], case["R"], t_range=(100, case["t_hi"]))]


def _sqn_data(case, seed):
    """Task 3's data (as workloads.sqn_dataset: sparse binary features, a random linear rule, 10%
    label noise), drawn on the GPU: (X uint8 [rows][n], z uint8 [rows])."""
    n, rows = case["n"], case["rows"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = min(0.5, 25.0 / n)
    a = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    X = torch.empty((rows, n), dtype=torch.uint8, device="cuda")
    z = torch.empty(rows, dtype=torch.uint8, device="cuda")
    for i in range(0, rows, 8192):
        x = torch.rand((min(8192, rows - i), n), generator=g, device="cuda") < p
        X[i:i + 8192] = x
        z[i:i + 8192] = (x.double() @ a) > p * a.sum()
    z ^= (torch.rand(rows, generator=g, device="cuda") < 0.1).to(torch.uint8)
    return X, z


def prepare(case, seed):
    s = dict(case=case, seed=seed, ctx=sim.Sim(0, torch.cuda.current_stream().cuda_stream))
    kind = case["kind"]
    if kind in ("paths", "dense", "latency", "cv", "wide"):
        kw = dict(N=case["N"], M=case.get("M", 1))
        if kind == "dense":
            kw["mu"], kw["chol"] = workloads.dense_instance(seed, 0, case["d"])
        else:
            kw["mu"], kw["sigma"] = _instance(case, seed, case["d"])
        if case.get("t_noise"):
            kw.update(noise=sim.NOISE_T, nu=3)
        kw["precision"] = sim.FP64 if case.get("fp64") else sim.FP32
        kw["checkpoints"] = (case["T"],) if kind in ("latency", "cv") else _ckpt(case["T"])
        s["problem"] = sim.Problem(keep_paths=case.get("keep", False), **kw)
    elif kind == "batch":
        s["problems"], s["T"] = [], []
        for i, (d, N, T) in enumerate(_sizes(case)):
            mu, sigma = _instance(case, seed, d, i)
            s["problems"].append(sim.Problem(mu=mu, sigma=sigma, N=N, instance_id=i))
            s["T"].append(T)
    elif kind in ("newsvendor", "lp"):
        s["inst"] = workloads.newsvendor_instance(seed, 0, case["n"])
        s["kw"] = dict(S=case["S"], M=case["M"], checkpoints=_ckpt(case["T"]))
        if kind == "lp":
            s["A"], s["C"] = workloads.newsvendor_constraints(seed, 0, case["n"], case["resources"])
    else:
        X, z = _sqn_data(case, seed)
        s["ctx"].sqn_load(X.cpu().numpy(), z.cpu().numpy())
        s["kw"] = dict(b=case["b"], bH=case["bH"], checkpoints=_ckpt(case["K"]), pairs_fp32=case["fp32"],
                       split=case["split"])
    return s


# ---- one pass ---------------------------------------------------------------------------------
def _stats(st, d=0):
    nc = st.n_checkpoints
    out = {f: float(getattr(st, f)) for f in ("mean", "var", "min", "max")}
    for f in ("f_mean", "f_sd", "rse_mean", "rse_sd"):
        out[f] = np.array(getattr(st, f)[:nc], dtype=np.float64)
    out["decision_total"] = np.array(st.decision_total[:d + 1], dtype=np.int64)
    out["tau_count"] = int(st.tau_count)
    return out


def run(s):
    case, ctx, seed, kind = s["case"], s["ctx"], s["seed"], s["case"]["kind"]
    if kind in ("paths", "dense"):
        ctx.run(s["problem"], case["R"], case["T"], seed)
        out = _stats(ctx.stats(), case["d"])
        if case.get("keep"):
            g = ctx.paths()
            out.update({k: g[k] for k in ("y", "f_ckpt", "cnt", "tau")})
            out["wsum"] = g["wsum"].astype(np.int64)
        return out
    if kind == "latency":
        ctx.run_batch([s["problem"]], [case["R"]], [case["T"]], seed, lanes_per_rep=[64], keep_paths=True)
        return dict(_stats(ctx.batch_stats(0), case["d"]), y=ctx.batch_paths(0)["y"])
    if kind == "batch":
        ctx.run_batch(s["problems"], [case["R"]] * case["n_inst"], s["T"], seed, keep_paths=True)
        sts = [_stats(ctx.batch_stats(i), 32) for i in range(case["n_inst"])]
        out = {f: np.array([st[f] for st in sts]) for f in ("mean", "var", "min", "max", "decision_total", "tau_count")}
        out["y"] = np.stack([ctx.batch_paths(i)["y"] for i in range(case["n_inst"])])
        return out
    if kind == "cv":
        fit = ctx.cv_fit(s["problem"], case["T"], seed, R_train=case["R_train"], R_pilot=case["R_train"],
                         epochs=case["epochs"], batch=case["batch"])
        st = ctx.run_cv(s["problem"], case["R"], case["T"], seed + 100, 4 * case["R"])
        out = {f: float(getattr(st, f)) for f in ("mean_plain", "var_plain", "mean_resid", "var_resid", "mean_h_aux",
                                                   "mean_cv", "var_est", "rho2")}
        out.update(theta=ctx.mlp_get_params(case["d"] + 2), beta=fit.beta, y_mean=fit.y_mean,
                   loss=fit.loss_last_epoch)
        return out
    if kind == "wide":
        ctx.run_wide(s["problem"], case["R"], case["T"], seed)
        st, g = ctx.wide_stats(), ctx.wide_paths()
    elif kind == "newsvendor":
        ctx.run_newsvendor(s["inst"], case["R"], case["T"], seed, **s["kw"])
        st, g = ctx.nv_stats(), ctx.nv_paths()
    elif kind == "lp":
        ctx.run_newsvendor_lp(s["inst"], s["A"], s["C"], case["R"], case["T"], seed, **s["kw"])
        st, g = ctx.nv_lp_stats(), ctx.nv_lp_paths()
        out = _stats(st)
        out.update({k: g[k] for k in ("y", "f_ckpt", "x", "tau", "basis", "value", "pivots")})
        return out
    else:
        ctx.run_sqn(case["R"], case["K"], seed, **s["kw"])
        out = _stats(ctx.sqn_stats())
        if not case["split"]:       # many replications: the loss statistics are the result
            return out
        g = ctx.sqn_paths()
        out.update({k: g[k] for k in ("F", "F_ckpt", "w", "pairs")})
        out["S"], out["Y"] = np.stack(g["S"]), np.stack(g["Y"])
        return out
    out = _stats(st)
    out.update({k: g[k] for k in ("y", "f_ckpt", "cnt", "tau", "decisions")})
    out["wsum"] = g["wsum"].astype(np.int64)
    return out


# ---- what the method cannot do without ----------------------------------------------------------
def _alg1_ops(R, T, d, N):
    return float(R) * T * (23.0 * N * d + 15.0 * d)


def work(case):
    kind = case["kind"]
    if kind in ("paths", "dense", "latency", "wide"):
        R, T, d = case["R"], case["T"], case["d"]
        ops = _alg1_ops(R, T, d, case["N"])
        if kind == "dense":                       # the products L'w and L h of every iteration
            ops += float(R) * T * 4.0 * d * d + (float(R) * T * case["N"] * 63.0 if case["t_noise"] else 0.0)
        nbytes = 16.0 * d + 8.0 * 5 * R
        if case.get("keep"):
            nbytes += R * (12.0 * d + 16)
        if kind == "wide":
            nbytes += 20.0 * R * d + 4.0 * R * T
        return dict(bytes=nbytes, flops=ops)
    if kind == "batch":
        return dict(bytes=8.0 * case["n_inst"] * case["R"], flops=sum(_alg1_ops(case["R"], T, d, N) for d, N, T in _sizes(case)))
    if kind == "cv":
        paths = 3 * case["R_train"] + case["R"]
        mlp = 2.0 * (64 * (case["d"] + 2) + 64 * 64 + 64)
        ops = _alg1_ops(paths, case["T"], case["d"], case["N"]) + mlp * (3.0 * case["epochs"] * case["R_train"] + 5.0 * case["R"])
        return dict(bytes=4.0 * (case["d"] + 3) * paths, flops=ops)
    if kind in ("newsvendor", "lp"):
        R, T, n = case["R"], case["T"], case["n"]
        out = 12.0 * R * n if kind == "newsvendor" else 8.0 * R * n + 12.0 * R * T * case["resources"]
        return dict(bytes=48.0 * n + out + 4.0 * R * T, flops=float(R) * T * n * (25.0 * case["S"] + 10.0))
    # SQN: the two passes over the stored pairs and the sampled rows' bits, every iteration
    n, K, R, L, M = case["n"], case["K"], case["R"], 10, 25
    steps = K // L
    held = sum(min(max(k // L - 1, 0), M) for k in range(1, K + 1))
    nbytes = R * (2.0 * 2 * 8 * n * held + K * (2.0 * case["b"] * n / 8 + 16 * n) + steps * (3.0 * case["bH"] * n / 8 + 24 * n))
    return dict(bytes=nbytes, flops=R * (8.0 * n * held + K * 100.0 * case["b"] + steps * 150.0 * case["bH"]))


# ---- 64-bit values by plain torch and numpy ------------------------------------------------------
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    lo32 = 0xFFFFFFFF
    k0, k1 = seed & lo32, (seed >> 32) & lo32
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2          # wraps modulo 2^64, which keeps both halves
        c0, c1, c2, c3 = ((p1 >> 32) & lo32) ^ c1 ^ k0, p1 & lo32, ((p0 >> 32) & lo32) ^ c3 ^ k1, p0 & lo32
        k0, k1 = (k0 + 0x9E3779B9) & lo32, (k1 + 0xBB67AE85) & lo32
    return c0, c1, c2, c3


def _normals(seed, word3, reps, epoch, q0, n):
    """Standard normals q0 .. q0+n-1 of the streams (reps, epoch): [len(reps)][n]."""
    b0, b1 = q0 // 4, (q0 + n + 3) // 4
    b = torch.arange(b0, b1, device="cuda", dtype=torch.int64)[None, :]
    r = reps[:, None]
    x = _philox(b.expand(len(reps), -1), torch.full_like(r, epoch), r, torch.full_like(r, word3), seed)
    u = [(2 * (w & 0x7FFFFF) + 1).double() * 2.0 ** -24 for w in x]
    out = []
    for u1, u2 in ((u[0], u[1]), (u[2], u[3])):
        rad = torch.sqrt(-2.0 * torch.log(u1))
        out += [rad * torch.cos(2.0 * math.pi * u2), rad * torch.sin(2.0 * math.pi * u2)]
    z = torch.stack(out, dim=2).reshape(len(reps), -1)
    return z[:, q0 - 4 * b0: q0 - 4 * b0 + n]


def _summary(y, f):
    """The floating statistics of outcomes y [R] and checkpoint values f [nc][R]."""
    out = dict(mean=float(y.mean()), min=float(y.min()), max=float(y.max()))
    if len(y) > 1:
        out["var"] = float(y.var(ddof=1))
    if len(f):
        rse = ((f - y) / f) ** 2
        out.update(f_mean=f.mean(1), rse_mean=rse.mean(1))
        if len(y) > 1:
            out.update(f_sd=f.std(1, ddof=1), rse_sd=rse.std(1, ddof=1))
    return out


def _alg1(mu, chol, N, M, R, T, seed, nu, checkpoints, instance=0):
    """Algorithm 1 in FP64: (y [R], f [nc][R]); chol a vector (diagonal) or a matrix."""
    mu, L = torch.tensor(mu, device="cuda"), torch.tensor(chol, device="cuda")
    d = len(mu)
    mult = (lambda v: v * L) if L.dim() == 1 else (lambda v: v @ L.T.contiguous())
    part = max(1, min(R, CHUNK // (N * (d + nu))))
    ys, fs = [], []
    for r0 in range(0, R, part):
        reps = torch.arange(r0, min(R, r0 + part), device="cuda", dtype=torch.int64)
        w = torch.zeros((len(reps), d), device="cuda", dtype=torch.float64)
        f = []

        def objective(w):
            v = w * L if L.dim() == 1 else w @ L
            return 0.5 * (v * v).sum(1) - w @ mu

        for t in range(T):
            if t % M == 0:
                z = _normals(seed, instance, reps, t // M, 0, N * (d + nu))
                if nu:
                    chi = z[:, N * d:].reshape(-1, N, nu).square().sum(2)
                    z = z[:, :N * d].reshape(-1, N, d) * torch.sqrt((nu - 2) / chi)[:, :, None]
                x = mult(z.reshape(-1, d)).reshape(-1, N, d)
                xbar = x.mean(1)
                x = x - xbar[:, None, :]
            g = ((x * w[:, None, :]).sum(2)[:, :, None] * x).sum(1) / (N - 1) - xbar - mu
            gmin, a = g.min(1)
            gamma = 2.0 / (t + 2)
            w = w * (1 - gamma)
            w[torch.arange(len(reps), device="cuda"), a] += gamma * (gmin < 0).double()
            if t + 1 in checkpoints:
                f.append(objective(w).cpu().numpy())
        ys.append(objective(w).cpu().numpy())
        fs.append(np.stack(f) if f else np.zeros((0, len(reps))))
    return np.concatenate(ys), np.concatenate(fs, axis=1)


def _nv_cost(p, x):
    z = (x - p["mu"]) / p["sigma"]
    pdf = torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)
    cdf, upper = 0.5 * torch.erfc(-z / math.sqrt(2)), 0.5 * torch.erfc(z / math.sqrt(2))
    return float((p["k"] * x + p["h"] * p["sigma"] * (z * cdf + pdf) + p["v"] * p["sigma"] * (pdf - z * upper)).sum())


def _simplex(g, A, C):
    """A vertex minimising g's over {A s <= C, s >= 0} (A >= 0), revised simplex from the slacks:
    (basic columns, values)."""
    m, n = A.shape
    basis, inv, xb = [n + i for i in range(m)], np.eye(m), C.copy()
    for _ in range(200):
        y = np.array([g[j] if j < n else 0.0 for j in basis]) @ inv
        rc = np.concatenate([g - y @ A, -y])
        q = int(np.argmin(rc))
        if rc[q] >= -1e-11:
            break
        dcol = inv @ (A[:, q] if q < n else np.eye(m)[:, q - n])
        ratio = np.where(dcol > 1e-12, xb / np.where(dcol > 1e-12, dcol, 1.0), np.inf)
        i = int(np.argmin(ratio))
        row = inv[i] / dcol[i]
        inv, xb = inv - np.outer(dcol, row), np.maximum(xb - dcol * ratio[i], 0.0)
        inv[i], xb[i], basis[i] = row, ratio[i], q
    return basis, xb


def _alg2(case, seed):
    inst = workloads.newsvendor_instance(seed, 0, case["n"])
    p = {f: torch.tensor(inst[f], device="cuda") for f in ("mu", "sigma", "k", "h", "v", "c")}
    n, S, M, lp = case["n"], case["S"], case["M"], case["kind"] == "lp"
    if lp:
        A, C = workloads.newsvendor_constraints(seed, 0, n, case["resources"])
    ys, fs, xs = [], [], []
    for r in range(case["R"]):
        rep = torch.tensor([r], device="cuda", dtype=torch.int64)
        x, f = torch.zeros(n, device="cuda", dtype=torch.float64), []
        for t in range(case["T"]):
            if t % M == 0:
                demand = p["mu"] + p["sigma"] * _normals(seed, 4 << 24, rep, t // M, 0, S * n).reshape(S, n)
            g = p["k"] - p["v"] + (p["h"] + p["v"]) * (demand <= x).double().sum(0) / S
            gamma = 2.0 / (t + 2)
            if lp:
                basis, xb = _simplex(g.cpu().numpy(), A, C)
                s = torch.zeros_like(x)
                for j, v in zip(basis, xb):
                    if j < n:
                        s[j] = v
                x = x + gamma * (s - x)
            else:
                ratio = g / p["c"]
                a = int(ratio.argmin())
                x = x * (1 - gamma)
                if float(ratio[a]) < 0:
                    x[a] += gamma * inst["C"] / float(p["c"][a])
            if t + 1 in _ckpt(case["T"]):
                f.append(_nv_cost(p, x))
        ys.append(_nv_cost(p, x))
        fs.append(f)
        xs.append(x.cpu().numpy())
    y, f = np.array(ys), np.array(fs).T.copy()
    out = dict(_summary(y, f), y=y, f_ckpt=f)
    if lp:
        out["x"] = np.stack(xs)
    return out


def _sqn(case, seed):
    n, rows, b, bH, K, L, M = case["n"], case["rows"], case["b"], case["bH"], case["K"], 10, 25
    X, z = _sqn_data(case, seed)
    zd = z.double()

    def indices(r, k, domain, count):
        q = torch.arange((count + 3) // 4, device="cuda", dtype=torch.int64)
        x = _philox(q, torch.full_like(q, k), torch.full_like(q, r), torch.full_like(q, domain << 24), seed)
        return ((torch.stack(x, 1).reshape(-1)[:count] * rows) >> 32)

    def loss(w):
        total = 0.0
        for i in range(0, rows, 16384):
            v = X[i:i + 16384].double() @ w
            total += float((torch.clamp(v, min=0) + torch.log1p(torch.exp(-v.abs())) - zd[i:i + 16384] * v).sum())
        return total / rows

    out = dict(F=[], F_ckpt=[], w=[], S=[], Y=[])
    for r in range(case["R"]):
        w = torch.zeros(n, device="cuda", dtype=torch.float64)
        acc, prev, pairs, f = torch.zeros_like(w), None, [], []
        for k in range(1, K + 1):
            i = indices(r, k, 5, b)
            x = X[i].double()
            g = (torch.sigmoid(x @ w) - zd[i]) @ x / b
            acc += w
            if k > 2 * L:                       # the two-loop form of Algorithm 4's matrix
                a = []
                for s, y, rho in reversed(pairs):
                    a.append(rho * (s @ g))
                    g = g - a[-1] * y
                s, y, rho = pairs[-1]
                g = g / (rho * (y @ y))
                for (s, y, rho), ai in zip(pairs, reversed(a)):
                    g = g + (ai - rho * (y @ g)) * s
            w = w - (2.0 / k) * g
            if k % L == 0:
                wbar = acc / L
                if prev is not None:
                    i = indices(r, k, 6, bH)
                    x = X[i].double()
                    c = torch.sigmoid(x @ wbar)
                    s = wbar - prev
                    y = (c * (1 - c) * (x @ s)) @ x / bH
                    pairs = (pairs + [(s, y, 1.0 / (s @ y))])[-M:]
                prev, acc = wbar, torch.zeros_like(w)
            if k in _ckpt(K):
                f.append(loss(w))
        out["F"].append(loss(w))
        out["F_ckpt"].append(f)
        out["w"].append(w.cpu().numpy())
        out["S"].append(np.stack([p[0].cpu().numpy() for p in pairs]))
        out["Y"].append(np.stack([p[1].cpu().numpy() for p in pairs]))
    out = {k: np.array(v) for k, v in out.items()}
    out["F_ckpt"] = out["F_ckpt"].T.copy()
    return dict(_summary(out["F"], out["F_ckpt"]), **out)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("paths", "dense", "latency", "wide"):
        R, T, d, N = case["R"], case["T"], case["d"], case["N"]
        parts = -(-R // max(1, min(R, CHUNK // (N * (d + 3)))))
        if float(R) * T * N * d > EXACT_NORMALS or float(T) * parts > 8000:
            return None
        mu, L = workloads.dense_instance(seed, 0, d) if kind == "dense" else _instance(case, seed, d)
        ck = (T,) if kind == "latency" else _ckpt(T)
        y, f = _alg1(mu, L, N, case.get("M", 1), R, T, seed, 3 if case.get("t_noise") else 0, ck)
        out = _summary(y, f)
        if kind in ("latency", "wide") or case.get("keep"):
            out["y"] = y
        if kind == "wide" or case.get("keep"):
            out["f_ckpt"] = f
        return out
    if kind == "batch":
        sizes = _sizes(case)
        if sum(float(case["R"]) * T * N * d for d, N, T in sizes) > EXACT_NORMALS or sum(T for _, _, T in sizes) > 8000:
            return None
        ys = []
        for i, (d, N, T) in enumerate(sizes):
            mu, sigma = _instance(case, seed, d, i)
            ys.append(_alg1(mu, sigma, N, 1, case["R"], T, seed, 0, (), i)[0])
        y = np.stack(ys)
        return dict(mean=y.mean(1), var=y.var(1, ddof=1), min=y.min(1), max=y.max(1), y=y)
    if kind in ("newsvendor", "lp"):
        if float(case["R"]) * case["T"] > 4000 or float(case["R"]) * case["T"] * case["n"] * case["S"] > EXACT_NORMALS:
            return None
        return _alg2(case, seed)
    if kind == "sqn":
        return _sqn(case, seed) if case["R"] * case["K"] <= 2000 and not case["fp32"] else None
    return None     # the control variate's network trains in bfloat16: no 64-bit value
