"""Performance cases: what a user of the framework has it do, through its
public entry points.

Kinds: the MD step loop of one channel and of batches of channels (with and
without the wall pressure), the statistics of sampled series, the GP
(fit, growth by new runs, dense maps, evidence search), the MLP ensemble
(training, dense maps) and the macro march.  Sizes come from `workloads`, the
benchmark and the studies: the 2,048-atom channel, the 39,189-atom channel, the
64-channel batch, density sweeps, 256 training runs, 48-run study databases,
databases up to the GP's 6144 points, 20,000-sample series.

Trajectory frames and logged series of the MD are kept in single precision,
as trajectory files are, and ensemble outputs in the networks' own precision.
"""
import math

import numpy as np
import torch

import paper_1603_04628_amd as hmd
from paper_1603_04628_amd import binding as B

BOX_SMALL, BOX_LARGE = 20.636, 57.146  # the 2,048-atom channel's box and the batch box
N_SAMPLE = 20000                       # sampled steps of the batch protocol
N_SHORT = 4000                         # sampled steps of a density sweep's run or a short fallback
RANGES = (16.0, 0.049)                 # spans of the channel heights and body forces


def listed():
    return [
        # one micro-solve of a small channel: the smallest MD step, launches and latency
        dict(name="channel_small", kind="md", channels=1, h_lo=6.0, h_hi=6.0, box=BOX_SMALL, n_fluid=2048, skin=0.3,
             pressure=0, steps=40),
        # one micro-solve of the paper-scale channel (39,189 atoms)
        dict(name="channel_paper", kind="md", channels=1, h_lo=15.0, h_hi=15.0, box=BOX_LARGE, n_fluid=0, skin=0.3,
             pressure=0, steps=40),
        # training batch of the benchmark: 64 uneven channels, 2.1 M atoms, tuned skin
        dict(name="batch_64", kind="md", channels=64, h_lo=4.0, h_hi=20.0, box=BOX_LARGE, n_fluid=0, skin=0.35,
             pressure=0, steps=40),
        # pre-simulations of the pressure surrogate: a density sweep with the wall pressure recorded
        dict(name="density_sweep", kind="md", channels=11, h_lo=6.0, h_hi=10.0, box=BOX_LARGE, n_fluid=0, skin=0.3,
             pressure=1, steps=40),
        # standard errors of a finished batch: 64 flux series of 20,000 samples
        dict(name="series_64", kind="series", S=64, n=N_SAMPLE, corr=1000.0),
        # one macro step of the march, 200 sections answered by the GP: the smallest call
        dict(name="march_step", kind="march", sections=200, points=256),
        # Alg. 1's database growth: 256 training runs, then a macro step's fallbacks one by one
        dict(name="gp_grow", kind="gp_grow", points=256, more=8, d=2, noise_mode=0),
        # fit near the upper end of the database sizes, (h, rho, F) inputs, each run's own noise
        dict(name="gp_fit_large", kind="gp_grow", points=3001, more=0, d=3, noise_mode=1),
        # a dense flux map from a grown database, on device tensors
        dict(name="gp_map", kind="gp_map", points=1000, queries=20000, d=2, noise_mode=0),
        # hyperparameters by the evidence on a study database (48 runs)
        dict(name="gp_evidence", kind="gp_evidence", points=48, d=2),
        # training of the 5-member ensemble on 256 runs
        dict(name="ens_fit", kind="ens_fit", points=256, members=5, hidden=64, iters=500, bootstrap=0),
        # a dense flux map from the ensemble, on device tensors
        dict(name="ens_map", kind="ens_map", points=256, members=5, hidden=64, queries=50000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["md", "md", "md", "series", "series", "march", "gp_grow", "gp_grow", "gp_map", "gp_evidence",
                       "ens_fit", "ens_map"])
    if kind == "md":
        many = rng.random() < 0.5
        h = round(rng.uniform(4.0, 20.0), 3)
        return dict(kind=kind, channels=_log(rng, 2, 24) if many else 1, h_lo=4.0 if many else h, h_hi=20.0 if many else h,
                    box=rng.choice([12.7, BOX_SMALL, 40.0, BOX_LARGE]), n_fluid=0, skin=rng.choice([0.3, 0.35]),
                    pressure=rng.choice([0, 0, 1]), steps=40)
    if kind == "series":
        return dict(kind=kind, S=_log(rng, 1, 64), n=_log(rng, 200, N_SAMPLE), corr=round(rng.uniform(20.0, 2000.0), 1))
    if kind == "march":
        return dict(kind=kind, sections=_log(rng, 5, 200), points=_log(rng, 16, 512))
    if kind == "gp_grow":
        n = _log(rng, 16, 3000)
        return dict(kind=kind, points=n, more=rng.randint(1, 8) if n <= 512 else 0, d=rng.randint(2, 3),
                    noise_mode=rng.randint(0, 1))
    if kind == "gp_map":
        n = _log(rng, 40, 1000)
        return dict(kind=kind, points=n, queries=_log(rng, 100, 20000), d=rng.randint(2, 3), noise_mode=rng.randint(0, 1))
    if kind == "gp_evidence":
        return dict(kind=kind, points=rng.randint(16, 48), d=rng.randint(2, 3))
    if kind == "ens_fit":
        return dict(kind=kind, points=_log(rng, 32, 256), members=rng.randint(2, 5), hidden=rng.choice([16, 32, 64]),
                    iters=rng.randint(100, 500), bootstrap=rng.randint(0, 1))
    return dict(kind=kind, points=_log(rng, 64, 256), members=rng.randint(2, 5), hidden=rng.choice([16, 32, 64]),
                queries=_log(rng, 200, 50000))


# ------------------------------------------------------------------ inputs
def _md_jobs(case, seed):
    """(h, g, seed, n_sample, rho) per channel, heights and forces of the batch ranges."""
    r = np.random.default_rng(seed)
    S = case["channels"]
    h = case["h_lo"] + (case["h_hi"] - case["h_lo"]) * ((np.arange(S) + r.uniform(0, 1, S)) / S if S > 1 else 0.0)
    h = np.broadcast_to(h, (S,))
    g = r.uniform(0.001, 0.05, S)
    rho = np.linspace(0.95, 0.7, S) if case["pressure"] else np.full(S, 0.8)
    n = N_SAMPLE if S == 1 else N_SHORT
    return [(float(h[k]), float(g[k]), int(seed) % 100000 + k, n, float(rho[k])) for k in range(S)]


def _extent(case):
    a = 4.0 ** (1.0 / 3.0)
    return max(1, round(case["box"] / a)) * a


def _channel_state(case, seed):
    """A start of one channel: atoms of a jittered simple lattice between the walls, Maxwell velocities."""
    h, _, _, _, rho = _md_jobs(case, seed)[0]
    L = _extent(case)
    n = case["n_fluid"] or int(math.floor(rho * L * L * h + 0.5))
    r = np.random.default_rng(seed + 1)
    best = None
    for ny in range(1, int((h - 2.0) / 0.5) + 2):
        nx = math.ceil(math.sqrt(n / ny))
        nz = math.ceil(n / (ny * nx))
        gap = min(L / nx, L / nz, (h - 2.0) / (ny - 1) if ny > 1 else L)
        if best is None or gap > best[0]:
            best = (gap, nx, ny, nz)
    _, nx, ny, nz = best
    s = np.sort(r.permutation(nx * ny * nz)[:n])
    x = np.stack([(s % nx + 0.5) * L / nx, 1.0 + (s // (nx * nz)) * ((h - 2.0) / max(ny - 1, 1)),
                  ((s // nx) % nz + 0.5) * L / nz], 1)
    if ny == 1:
        x[:, 1] = 0.5 * h
    x += r.uniform(-0.02, 0.02, x.shape)
    v = r.standard_normal((n, 3))
    v -= v.mean(0)
    return x, v / math.sqrt((v * v).mean())


def _series(case, seed):
    """Flux-like series: a slowly decaying, a fast and a white part about a mean."""
    r = np.random.default_rng(seed)
    S, n = case["S"], case["n"]
    m = 2 * n
    f = np.fft.rfftfreq(m)
    out = np.zeros((S, n))
    for amp, tau in ((1.0, case["corr"]), (0.5, 12.0)):
        a = math.exp(-1.0 / tau)
        z = np.fft.irfft(np.fft.rfft(r.standard_normal((S, m)), axis=1) / (1.0 - a * np.exp(-2j * np.pi * f)), m, axis=1)
        out += amp * math.sqrt(1.0 - a * a) * z[:, :n]
    return np.ascontiguousarray(0.3 + 0.05 * (out + 0.2 * r.standard_normal((S, n))))


def _points(n, d, seed):
    """A flux database: inputs over the batch ranges, a smooth law, the runs' noise and standard errors."""
    r = np.random.default_rng(seed)
    h, g, rho = r.uniform(4.0, 20.0, n), r.uniform(0.001, 0.05, n), r.uniform(0.7, 0.95, n)
    y = 0.002 * h ** 3 * g * (1.0 + 0.2 * np.sin(h)) * (1.0 if d == 2 else 1.8 - rho)
    se = r.uniform(0.005, 0.02, n)
    y = y + se * r.standard_normal(n)
    X = np.stack([h, g], 1) if d == 2 else np.stack([h, rho, g], 1)
    return np.ascontiguousarray(X), y, se


def _hyper(case):
    d3 = case.get("d", 2) == 3
    return dict(sigma_f=3.0, ell=2.0, ranges=(16.0, 0.25, 0.049) if d3 else RANGES, noise_mode=case.get("noise_mode", 0))


def _march(case):
    """Macro constants: converging-diverging channel, pressure drop from the throat force, explicit macro step."""
    n, L = case["sections"], 10.0 * case["sections"]
    h = 10.0 * (1.0 + 0.5 * np.cos(2.0 * np.pi * (np.arange(n) + 0.5) / n))
    c = 0.038 * 125.0
    return dict(n_sections=n, h0=10.0, amp=0.5, L=L, rho_ref=0.8, p_out=0.0, dp_mean=0.8 * c * float((h ** -3.0).sum()) * 10.0,
                dp_amp=0.1, period=250.0, c2=200.0, dt_macro=0.1, tau_rel=0.0, tau_abs=1e9, surrogate=0)


def _march_start(case, seed):
    m = _march(case)
    r = np.random.default_rng(seed + 5)
    frac = 1.0 - (np.arange(case["sections"]) + 0.5) / case["sections"]
    return 0.8 + m["dp_mean"] * frac / m["c2"] + r.uniform(-1e-4, 1e-4, case["sections"])


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    kind = case["kind"]
    if kind == "md":
        ctx = hmd.Context(hmd.Params(Lx_nom=case["box"], Lz_nom=case["box"], n_fluid=case["n_fluid"], skin=case["skin"],
                                     pressure=case["pressure"]))
        b = hmd.Batch(ctx, _md_jobs(case, seed))
        if case["channels"] == 1:
            b.set_state(0, *_channel_state(case, seed))
        return dict(case=case, ctx=ctx, batch=b)
    ctx = hmd.Context(hmd.Params(Lx_nom=BOX_LARGE, Lz_nom=BOX_LARGE))
    st = dict(case=case, ctx=ctx)
    if kind in ("series", "gp_map", "ens_map"):
        st["stream"] = torch.cuda.Stream()  # the calls on device tensors run on the program's own stream
    if kind == "series":
        st["x"] = torch.from_numpy(_series(case, seed)).cuda()
    elif kind == "march":
        gp = hmd.GP(ctx, *_points(case["points"], 2, seed), B.gp_hyper(**_hyper(case)))
        st["hy"] = hmd.Hybrid(ctx, hmd.hybrid_cfg(**_march(case)), gp=gp)
        st["hy"].set_rho(_march_start(case, seed))
    elif kind in ("gp_grow", "gp_evidence"):
        st["data"] = _points(case["points"] + case.get("more", 0), case["d"], seed)
        st["q"] = _points(200, case["d"], seed + 77)[0]
    elif kind == "gp_map":
        st["gp"] = hmd.GP(ctx, *_points(case["points"], case["d"], seed), B.gp_hyper(**_hyper(case)))
        st["q"] = torch.from_numpy(_points(case["queries"], case["d"], seed + 77)[0]).cuda()
    elif kind == "ens_fit":
        st["data"] = _points(case["points"], 2, seed)
        st["q"] = _points(200, 2, seed + 77)[0]
    elif kind == "ens_map":
        X, y, _ = _points(case["points"], 2, seed)
        st["ens"] = hmd.Ensemble(ctx, X, y, hmd.ens_cfg(members=case["members"], hidden=case["hidden"], iters=200))
        st["q"] = torch.from_numpy(_points(case["queries"], 2, seed + 77)[0]).cuda()
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "md":
        # a segment of the run, then its log: the flux (and pressure) series so
        # far, the energies, and the frame of a single channel
        b = state["batch"]
        b.run(case["steps"], case["steps"])
        out = dict(flux=np.stack([b.series(k) for k in range(b.n)]).astype(np.float32),
                   pe=np.array([r["pe"] for r in b.results()], dtype=np.float32))
        if case["pressure"]:
            out["p"] = np.stack([b.pressure_series(k) for k in range(b.n)]).astype(np.float32)
        if b.n == 1:
            x, v = b.get_state(0)
            out["x"], out["v"] = x.astype(np.float32), v.astype(np.float32)
        return out
    if kind == "series":
        with torch.cuda.stream(state["stream"]):
            return B.series_stats_dev(state["ctx"], state["x"])
    if kind == "march":
        state["hy"].step()
        return state["hy"].get()
    if kind == "gp_grow":
        X, y, se = state["data"]
        n = case["points"]
        gp = hmd.GP(state["ctx"], X[:n], y[:n], se[:n], B.gp_hyper(**_hyper(case)))
        for k in range(n, n + case["more"]):
            gp.append(X[k], y[k], se[k])
        mean, var = gp.predict(state["q"])
        out = dict(mean=mean, var=var, lml=gp.log_marginal())
        gp.close()
        return out
    if kind == "gp_map":
        with torch.cuda.stream(state["stream"]):
            mean, var = state["gp"].predict_dev(state["q"])
        return dict(mean=mean, var=var)
    if kind == "gp_evidence":
        gp = hmd.GP(state["ctx"], *state["data"], B.gp_hyper(ranges=_hyper(case)["ranges"]))
        lml = gp.optimize(("sigma_f", "ell"))
        hp = gp.hyper()
        gp.close()
        return dict(lml=lml, sigma_f=hp["sigma_f"], ell=hp["ell"])
    if kind == "ens_fit":
        X, y, _ = state["data"]
        e = hmd.Ensemble(state["ctx"], X, y, hmd.ens_cfg(members=case["members"], hidden=case["hidden"],
                                                         iters=case["iters"], bootstrap=case["bootstrap"]))
        mean, std = e.predict(state["q"])
        out = dict(mean=mean.astype(np.float32), std=std.astype(np.float32), loss=e.losses().astype(np.float32))
        e.close()
        return out
    with torch.cuda.stream(state["stream"]):
        mean, std = state["ens"].predict_dev(state["q"])
        return dict(mean=mean.float(), std=std.float())


def work(case):
    kind = case["kind"]
    if kind == "md":
        # in-cutoff pairs of the full neighbour sum at 27 operations, the state read and written once a pass
        L, S = _extent(case), case["channels"]
        atoms = case["n_fluid"] or 0.8 * L * L * 0.5 * (case["h_lo"] + case["h_hi"]) * S
        return dict(bytes=atoms * 96.0, flops=case["steps"] * atoms * (27.0 * 56.0 + 30.0))
    if kind == "series":
        # lags up to a few correlation times enter the estimator
        lags = min(case["n"], 6.0 * case["corr"])
        return dict(bytes=8.0 * case["S"] * case["n"], flops=2.0 * case["S"] * case["n"] * lags)
    if kind == "ens_fit":
        p = case["hidden"] * (case["hidden"] + 5) + 1
        return dict(bytes=4.0 * p * case["members"], flops=6.0 * p * case["points"] * case["members"] * case["iters"])
    if kind == "ens_map":
        p = case["hidden"] * (case["hidden"] + 5) + 1
        return dict(bytes=case["queries"] * 32.0, flops=2.0 * p * case["members"] * case["queries"])
    n = case["points"]
    if kind == "march":
        return dict(bytes=4.0 * n * n, flops=case["sections"] * (n * (n + 12.0)))
    if kind == "gp_map":
        return dict(bytes=4.0 * n * n + 40.0 * case["queries"], flops=case["queries"] * n * (n + 12.0))
    if kind == "gp_evidence":
        return dict(bytes=40.0 * n, flops=(289 + 1000) * (n ** 3 / 3.0 + 8.0 * n * n))  # grid and line searches
    return dict(bytes=40.0 * n, flops=(1 + case["more"]) * (n ** 3 / 3.0) + 200.0 * n * n)


# ------------------------------------------------------------------ 64-bit results
def exact(case, seed):
    kind = case["kind"]
    if kind == "md":
        return _exact_channel(case, seed) if case["channels"] == 1 else None  # whole batches take minutes
    if kind == "series":
        return _exact_series(_series(case, seed))
    if kind == "gp_evidence":
        return _exact_evidence(case, seed)
    if kind == "ens_fit" or kind == "ens_map":
        return _exact_ensemble(case, seed)
    if kind == "march":
        return _exact_march(case, seed)
    n = case["points"] + case.get("more", 0)
    X, y, se = _points(n, case["d"], seed)
    Q = _points(200 if kind == "gp_grow" else case["queries"], case["d"], seed + 77)[0]
    mean, var, lml = _gp64(X, y, se, Q, case.get("noise_mode", 0), 3.0, 2.0)
    return dict(mean=mean, var=var, lml=lml) if kind == "gp_grow" else dict(mean=mean, var=var)


def _t(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float64, device="cuda" if torch.cuda.is_available() else "cpu")


def _mean_separation(X):
    X = _t(X)
    n = len(X)
    return torch.stack([(X[:, None, k] - X[None, :, k]).abs().sum() / (n * (n - 1)) for k in range(X.shape[1])])


def _gp64(X, y, se, Q, noise_mode, sigma_f, ell):
    sc = _mean_separation(X)
    s_q = math.sqrt(float((y * y).mean()))
    noise = _t(se / s_q) if noise_mode else _t(np.full(len(y), se.mean() / s_q))
    A, q, t = _t(X) / sc, _t(Q) / sc, _t(y / s_q)

    def cov(a, b):
        return sigma_f ** 2 * torch.exp(-sum((a[:, None, k] - b[None, :, k]) ** 2 for k in range(a.shape[1])) / (2 * ell * ell))
    L = torch.linalg.cholesky(cov(A, A) + torch.diag(noise * noise))
    alpha = torch.cholesky_solve(t[:, None], L)[:, 0]
    mean, var = [], []
    for c in q.split(5000):
        K = cov(A, c)
        mean.append(K.T @ alpha)
        var.append(sigma_f ** 2 - (torch.linalg.solve_triangular(L, K, upper=False) ** 2).sum(0))
    lml = -0.5 * float(t @ alpha) - float(L.diagonal().log().sum()) - 0.5 * len(y) * math.log(2 * math.pi)
    return torch.cat(mean) * s_q, torch.cat(var) * s_q ** 2, lml


def _exact_evidence(case, seed):
    """The evidence's maximum over (log sigma_f, log ell) within two decades: a grid, then ever finer grids."""
    X, y, se = _points(case["points"], case["d"], seed)
    s_q = math.sqrt(float((y * y).mean()))
    A, t, sn2 = _t(X) / _mean_separation(X), _t(y / s_q), (se.mean() / s_q) ** 2
    d2 = sum((A[:, None, k] - A[None, :, k]) ** 2 for k in range(A.shape[1]))
    eye = torch.eye(len(y), dtype=torch.float64, device=d2.device)

    def lml(lf, ll):
        C = torch.exp(2 * lf)[:, None, None] * torch.exp(-d2 / (2 * torch.exp(2 * ll)[:, None, None])) + sn2 * eye
        L, bad = torch.linalg.cholesky_ex(C)
        z = torch.linalg.solve_triangular(L, t[None, :, None].expand(len(C), -1, 1), upper=False)[..., 0]
        f = -0.5 * (z * z).sum(1) - L.diagonal(dim1=1, dim2=2).log().sum(1) - 0.5 * len(y) * math.log(2 * math.pi)
        return torch.where((bad == 0) & f.isfinite(), f, torch.full_like(f, -math.inf))
    c, w, n = _t([0.0, 0.0]), 2 * math.log(10.0), 17
    for _ in range(40):
        u = torch.linspace(-w, w, n, dtype=torch.float64, device=d2.device)
        lf, ll = (c[0] + u).repeat_interleave(n), (c[1] + u).repeat(n)
        f = lml(lf, ll)
        k = int(f.argmax())
        c, w = torch.stack([lf[k], ll[k]]), w * 0.5 if w < 0.5 else w * 0.25
    return dict(lml=float(lml(c[:1], c[1:])[0]), sigma_f=float(c[0].exp()), ell=float(c[1].exp()))


def _exact_march(case, seed):
    m, n = _march(case), case["sections"]
    h = 10.0 * (1.0 + 0.5 * np.cos(2.0 * np.pi * (np.arange(n) + 0.5) / n))
    rho = _march_start(case, seed)
    p = np.concatenate([[m["dp_mean"]], m["c2"] * (rho - 0.8), [0.0]])
    g = -(p[2:] - p[:-2]) / 20.0 / rho
    X, y, se = _points(case["points"], 2, seed)
    mean, var, _ = _gp64(X, y, se, np.stack([h, np.abs(g)], 1), 0, 3.0, 2.0)
    q = np.sign(g) * mean.cpu().numpy()
    face = np.concatenate([q[:1], 0.5 * (q[1:] + q[:-1]), q[-1:]])
    return dict(rho=(rho * h - m["dt_macro"] * np.diff(face) / 10.0) / h, q=q, g=g, from_md=None,
                q_std=np.sqrt(np.maximum(var.cpu().numpy(), 0.0)))


def _exact_series(x):
    S, n = x.shape
    mean = x.mean(1)
    F = np.fft.rfft(x - mean[:, None], 2 * n, axis=1)
    gam = np.fft.irfft(F * F.conj(), 2 * n, axis=1)[:, :n] / n
    out = np.stack([mean, np.zeros(S), x[:, :n // 2].mean(1), x[:, n // 2:].mean(1)], 1)
    for s in range(S):
        pair = gam[s, 0:2 * (n // 2):2] + gam[s, 1:2 * (n // 2):2]
        stop = int(np.argmax(pair <= 0.0)) if (pair <= 0.0).any() else len(pair)
        var = -gam[s, 0] + 2.0 * np.minimum.accumulate(pair[:stop]).sum() if stop else gam[s, 0]
        out[s, 1] = math.sqrt((var if var > 0.0 else gam[s, 0]) / n)
    return out


def _philox(ctr, key):
    """Philox4x32-10 for an (m, 4) array of counters."""
    c = [ctr[:, k].astype(np.uint64) for k in range(4)]
    k0, k1 = key
    lo = np.uint64(0xffffffff)
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & lo, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & lo]
        k0, k1 = (k0 + 0x9E3779B9) & 0xffffffff, (k1 + 0xBB67AE85) & 0xffffffff
    return np.stack(c, 1)


def _exact_ensemble(case, seed):
    """The members trained in 64 bits.  Their spread and final loss are small differences that the 32-bit training
    itself leaves uncertain, so only the mean has a value."""
    X, y, _ = _points(case["points"], 2, seed)
    fit = case["kind"] == "ens_fit"
    Q = _points(200 if fit else case["queries"], 2, seed + 77)[0]
    H, M, n = case["hidden"], case["members"], case["points"]
    mu, sd, s_q = X.mean(0), X.std(0), math.sqrt(float((y * y).mean()))
    x, q, t = (_t(a.astype(np.float32)) for a in ((X - mu) / sd, (Q - mu) / sd, y / s_q))
    P = H * H + 5 * H + 1
    th, wt = [], []
    for k in range(M):
        j = np.arange((P + 3) // 4)
        u = (_philox(np.stack([j, j * 0 + k, j * 0 + 2, j * 0], 1), (0, 0)).reshape(-1)[:P] + 0.5) / 2.0 ** 32
        lim = np.zeros(P)
        lim[:2 * H], lim[3 * H:3 * H + H * H], lim[4 * H + H * H:5 * H + H * H] = (math.sqrt(6 / a) for a in (2.0 + H, 2.0 * H, H + 1.0))
        th.append((lim * (2 * u - 1)).astype(np.float32))
        j = np.arange((n + 3) // 4)
        r = _philox(np.stack([j, j * 0 + k, j * 0 + 3, j * 0], 1), (0, 0)).reshape(-1)[:n]
        wt.append(np.bincount(((r * np.uint64(n)) >> np.uint64(32)).astype(np.int64), minlength=n) if case.get("bootstrap") else np.ones(n))
    th, w = _t(np.stack(th)), _t(np.stack(wt))

    def net(p, z):
        W1, b1, W2, b2, W3, b3 = p.split([2 * H, H, H * H, H, H, 1], 1)
        h1 = torch.tanh(z[None] @ W1.view(M, H, 2).mT + b1[:, None])
        h2 = torch.tanh(h1 @ W2.view(M, H, H).mT + b2[:, None])
        return (h2 @ W3.view(M, H, 1))[..., 0] + b3
    m, v = torch.zeros_like(th), torch.zeros_like(th)
    for it in range(1, (case["iters"] if fit else 200) + 1):
        p = th.detach().requires_grad_()
        r = net(p, x) - t
        g, = torch.autograd.grad((w * r * r).sum() / n, p)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        th = th - 1e-3 * (m / (1 - 0.9 ** it)) / (torch.sqrt(v / (1 - 0.999 ** it)) + 1e-8)
    out = dict(mean=net(th, q).mean(0) * s_q, std=None)
    return dict(out, loss=None) if fit else out


def _exact_channel(case, seed):
    """Velocity Verlet, Berendsen on v_y and the shifted Lennard-Jones forces of one channel in 64 bits."""
    h, g, _, _, _ = _md_jobs(case, seed)[0]
    x, v = (_t(a) for a in _channel_state(case, seed))
    dev, n, L, rc, dt, steps = x.device, len(x), _extent(case), 2.5, 0.005, case["steps"]
    half = 0.5 * 4.0 ** (1.0 / 3.0)
    c = round(L / half)
    wall = []
    for k in range(4):
        pq = torch.cartesian_prod(torch.arange(c), torch.arange(c))
        pq = pq[(pq.sum(1) + k) % 2 == 0].double() * half
        wall += [torch.stack([pq[:, 0], torch.full((len(pq),), y, dtype=torch.float64), pq[:, 1]], 1) for y in (-k * half, h + k * half)]
    wall = torch.cat(wall).to(dev)
    box = torch.tensor([L, 0.0, L], dtype=torch.float64, device=dev)
    shift = 4.0 * (rc ** -12.0 - rc ** -6.0)

    def near(x):
        """Pairs (fluid atom, any other atom) within rc + 0.8."""
        every, ii, jj = torch.cat([x, wall]), [], []
        for a in range(0, n, 1024):
            d2 = torch.zeros(min(1024, n - a), len(every), dtype=torch.float64, device=dev)
            for k in range(3):
                d = x[a:a + 1024, k, None] - every[None, :, k]
                d2 += (d - L * torch.round(d / L) if k != 1 else d) ** 2
            i, j = (d2 < (rc + 0.8) ** 2).nonzero(as_tuple=True)
            keep = i + a != j
            ii.append(i[keep] + a)
            jj.append(j[keep])
        return torch.cat(ii), torch.cat(jj)

    def forces(x, i, j):
        d = x[i] - torch.cat([x, wall])[j]
        d[:, 0::2] -= L * torch.round(d[:, 0::2] / L)
        r2 = (d * d).sum(1)
        s6 = torch.where(r2 < rc * rc, r2 ** -3.0, torch.zeros_like(r2))
        f = torch.zeros_like(x).index_add_(0, i, (24.0 * s6 * (2.0 * s6 - 1.0) / r2)[:, None] * d)
        u = torch.where(s6 > 0, 4.0 * s6 * (s6 - 1.0) - shift, torch.zeros_like(s6)) * torch.where(j < n, 0.5, 1.0)
        lower = (j >= n) & (d[:, 1] > 0)
        fy = (24.0 * s6 * (2.0 * s6 - 1.0) / r2) * d[:, 1]
        press = 0.5 * (fy[lower].sum() - fy[(j >= n) & (d[:, 1] < 0)].sum()) / (L * L)
        return f, u.sum(), press

    i, j = near(x)
    x0 = x.clone()
    f, _, _ = forces(x, i, j)
    q, ps = torch.zeros(N_SAMPLE, dtype=torch.float64), torch.zeros(N_SAMPLE, dtype=torch.float64)
    push = torch.tensor([g, 0.0, 0.0], dtype=torch.float64, device=dev)
    for s in range(steps):
        v = v + 0.5 * dt * (f + push)
        x = x + dt * v
        x[:, 0::2] = torch.remainder(x[:, 0::2], L)
        d = x - x0
        d[:, 0::2] -= L * torch.round(d[:, 0::2] / L)
        if float((d * d).sum(1).max()) > 0.39 ** 2:
            i, j = near(x)
            x0 = x.clone()
        f, pe, press = forces(x, i, j)
        v = v + 0.5 * dt * (f + push)
        q[s], ps[s] = v[:, 0].sum() / (L * L), press
        v[:, 1] *= torch.sqrt(1.0 + dt / 0.1 * (1.0 / (v[:, 1] ** 2).mean() - 1.0))
    out = dict(flux=q[None], pe=pe[None] / n, x=x, v=v)
    return dict(out, p=ps[None]) if case["pressure"] else out
