"""Mean and standard error of sampled flux series on the device, against the
oracle's estimator (Sec. 2.3: the noise of an MD run is the standard deviation
of its mean, estimated from the raw time-instantaneous data), and the per-step
flux series of the MD path against the oracle's from one identical state.

Bars: the device statistics of a given series equal the oracle's to 1e-10
relative (FP64 sums in another order); the per-step flux from identical states
differs only by FP32 force rounding; the SE a run reports is the oracle's
estimator applied to that run's own series.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

hmd = pytest.importorskip("paper_1603_04628_amd")
from paper_1603_04628_amd import binding as B  # noqa: E402
from oracle import md as omd  # noqa: E402
from oracle import stats as ostats  # noqa: E402
import workloads  # noqa: E402

SMALL_L = dict(Lx_nom=workloads.BOX_SMALL_LITERAL, Lz_nom=workloads.BOX_SMALL_LITERAL)


def _ar1(seed, phi, n):
    rng = np.random.default_rng(seed)
    e = rng.standard_normal(n)
    x = np.empty(n)
    x[0] = e[0] / np.sqrt(1.0 - phi * phi)
    for t in range(1, n):
        x[t] = phi * x[t - 1] + e[t]
    return 0.3 + 0.01 * x


@pytest.mark.parametrize("S,n,rho", [(1, 112, 0.9), (1, 113, 0.9), (3, 224, 0.999), (64, 5000, 0.9995),
                                     (600, 304, 0.99), (600, 305, 0.99), (2, 6001, 0.9999)])
def test_lag_tiles_and_batches_match_oracle(S, n, rho):
    # around the lag tiles of both sizes (112, 304) and over several batches of
    # lags (long correlations: rows end in different batches); FP64 sums of n
    # products in another order: 1e-12 of gamma_0, which a variance that is a
    # sum of like terms keeps to 1e-9
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    rows = np.stack([_ar1(100 + k, rho * (0.5 + 0.5 * ((k % 7) / 6)), n) for k in range(S)])
    out = B.series_stats(ctx, rows)
    for k in range(S):
        m, se = ostats.geyer(rows[k])
        assert out[k, 0] == pytest.approx(m, rel=1e-12, abs=1e-14)
        assert out[k, 1] == pytest.approx(se, rel=1e-9)


@pytest.mark.parametrize("S,n", [(200, 511), (200, 512), (204, 600), (205, 600), (255, 513), (256, 513), (300, 575),
                                 (300, 576), (300, 577), (3, 1023), (3, 1025), (3, 1087), (3, 1088), (3, 1135),
                                 (9, 1136), (40, 2049)])
def test_rows_that_end_inside_a_pass_match_oracle(S, n):
    # ends of the last pass of 1,024 samples around whole steps of 64, on both
    # sides of the choice of tiles and of their batches; bars of
    # test_lag_tiles_and_batches_match_oracle
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    rows = np.stack([_ar1(300 + k, (0.0, 0.9, 0.998)[k % 3], n) for k in range(S)])
    out = B.series_stats(ctx, rows)
    for k in sorted({0, 1, 2, S // 2, S - 1}):
        m, se = ostats.geyer(rows[k])
        assert out[k, 0] == pytest.approx(m, rel=1e-12, abs=1e-14)
        assert out[k, 1] == pytest.approx(se, rel=1e-9)


@pytest.mark.parametrize("S,n", [(1, 2), (5, 3), (4, 63), (4, 64), (4, 65), (9, 128), (2, 256), (2, 257), (1023, 511),
                                 (1024, 512), (1024, 513)])
def test_short_rows_match_oracle(S, n):
    # both sides of the lengths a wavefront takes alone (256 for few rows, 512
    # for many), runs of 64 lags and their ends; bars of
    # test_lag_tiles_and_batches_match_oracle.  Rows stop in every run of lags
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    rows = np.stack([_ar1(300 + k, (0.0, 0.9, 0.99, 1.0 - 1e-6)[k % 4], n) for k in range(S)])
    out = B.series_stats(ctx, rows)
    for k in range(0, S, max(1, S // 64)):
        m, se = ostats.geyer(rows[k])
        h1, h2 = ostats.halves(rows[k])
        assert out[k, 0] == pytest.approx(m, rel=1e-12, abs=1e-14)
        assert out[k, 1] == pytest.approx(se, rel=1e-9)
        assert out[k, 2] == pytest.approx(h1, rel=1e-12, abs=1e-14)
        assert out[k, 3] == pytest.approx(h2, rel=1e-12, abs=1e-14)


def test_short_rows_of_unusual_values():
    # a constant row has no error; a row that holds a NaN or an infinity gives
    # NaN and leaves its neighbours alone
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    rows = np.stack([_ar1(1, 0.5, 100)] * 6)
    rows[1] = 0.25
    rows[2, 40] = np.nan
    rows[4, 99] = np.inf
    out = B.series_stats(ctx, rows)
    m, se = ostats.geyer(rows[0])
    for k in (0, 3, 5):
        assert out[k, 0] == pytest.approx(m, rel=1e-12) and out[k, 1] == pytest.approx(se, rel=1e-9)
    assert out[1, 0] == 0.25 and out[1, 1] == 0.0
    assert np.isnan(out[2, :2]).all() and np.isnan(out[4, 1]) and np.isinf(out[4, 0])


@pytest.mark.parametrize("n", [2, 3, 257, 1000, 20000])
def test_series_stats_match_oracle(n):
    # four rows (iid, short and long correlation, anti-correlated) in one call;
    # lengths below, at and across the 256-lag tiles, ragged tails included
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    rows = np.stack([_ar1(1, 0.0, n), _ar1(2, 0.9, n), _ar1(3, 0.995, n), _ar1(4, -0.5, n)])
    out = B.series_stats(ctx, rows)
    for k, r in enumerate(rows):
        m, se = ostats.geyer(r)
        h1, h2 = ostats.halves(r)
        assert out[k, 0] == pytest.approx(m, rel=1e-12)
        assert out[k, 1] == pytest.approx(se, rel=1e-10), (k, out[k, 1], se)
        assert out[k, 2] == pytest.approx(h1, rel=1e-12)
        assert out[k, 3] == pytest.approx(h2, rel=1e-12)
    if n >= 20:
        outb = B.series_stats(ctx, rows, n_blocks=20)
        for k, r in enumerate(rows):
            m, se = ostats.blocks(r, 20)
            assert outb[k, 0] == pytest.approx(m, rel=1e-12)
            assert outb[k, 1] == pytest.approx(se, rel=1e-10)


def test_series_stats_row_stride_and_dev_form():
    import torch
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    rows = np.stack([_ar1(7 + k, 0.8, 3001) for k in range(3)])
    host = B.series_stats(ctx, rows)
    dev = B.series_stats_dev(ctx, torch.from_numpy(rows).cuda())
    torch.cuda.synchronize()
    assert np.allclose(dev.cpu().numpy(), host, rtol=1e-14, atol=0)
    # a larger call after a smaller one grows the context's scratch
    big = np.stack([_ar1(20 + k, 0.95, 6000) for k in range(5)])
    dev2 = B.series_stats_dev(ctx, torch.from_numpy(big).cuda())
    torch.cuda.synchronize()
    for k, r in enumerate(big):
        assert dev2[k, 1].item() == pytest.approx(ostats.geyer(r)[1], rel=1e-10)


def test_series_stats_rejects_bad_sizes():
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    with pytest.raises(hmd.HmdError):
        B.series_stats(ctx, np.zeros(1))
    with pytest.raises(hmd.HmdError):
        B.series_stats(ctx, np.zeros(10), n_blocks=20)
    with pytest.raises(hmd.HmdError):
        B.series_stats(ctx, np.zeros(10), n_blocks=1)


@pytest.mark.parametrize("path", [0, 1, 2])
def test_flux_series_from_identical_state(path):
    # Sec. 2.1: every sampled step gives q' = sum(m v_x) / (Lx Lz).  From one
    # equilibrated state, 60 sampled steps on each side differ only by FP32
    # force rounding: each step's q' agrees far below the scale of the sum
    # (sum |v_x| / (Lx Lz)), which pins the normalisation and the step index
    pre = omd.System(6.0, 0.05, 7, omd.Params(**SMALL_L))
    pre.run(300)
    x, v = pre.get_state()
    n = 60
    params = dict(n_equil=0, **SMALL_L)
    ora = omd.System(6.0, 0.05, 7, omd.Params(cell_w=2.8 if path else 0.0, **params))
    ora.set_state(x, v)
    ora.run(n)
    qo = ora.series()
    ctx = hmd.Context(hmd.Params(force_path=path, skin=0.3, **params))
    b = hmd.Batch(ctx, [(6.0, 0.05, 7, n)])
    b.set_state(0, x, v)
    b.run(n, graph_chunk=20)
    qg = b.series(0)
    assert len(qg) == n == len(qo)
    scale = np.abs(v[:, 0]).sum() / (ora.Lx * ora.Lz)
    assert np.abs(qg - qo).max() <= 1e-6 * scale, np.abs(qg - qo).max() / scale
    # the first step's q' follows from the given velocities and forces alone
    assert abs(qg[0] - qo[0]) <= 1e-7 * scale
    r = b.results()[0]
    ro = ora.result()
    assert r["status"] == 0 and ro["status"] == 0
    assert r["flux"] == pytest.approx(ro["flux"], abs=1e-6 * scale)
    assert r["T"][1] == pytest.approx(ro["T"][1], rel=1e-5)


def test_results_se_is_the_oracle_estimator_of_the_run_series():
    # the SE a run reports is Geyer's estimator of its own series, exactly
    params = dict(n_equil=200, **SMALL_L)
    ctx = hmd.Context(hmd.Params(**params))
    jobs = [(6.0, 0.05, 3, 3000), (4.5, 0.02, 4, 3000), (9.0, 0.01, 5, 3000)]
    b = hmd.Batch(ctx, jobs)
    b.run(3200, graph_chunk=100)
    res = b.results()
    for k, r in enumerate(res):
        q = b.series(k)
        m, se = ostats.geyer(q)
        h1, h2 = ostats.halves(q)
        assert r["flux"] == pytest.approx(m, rel=1e-12)
        assert r["flux_se"] == pytest.approx(se, rel=1e-9)
        assert r["status"] in (0, -5)
        if r["status"] == -5:
            assert abs(h2 - h1) > 8.0 * se


def test_incomplete_window_is_not_a_result():
    # results before every sampling step has run carry HMD_EINVAL
    ctx = hmd.Context(hmd.Params(n_equil=50, **SMALL_L))
    b = hmd.Batch(ctx, [(6.0, 0.02, 1, 101)])
    b.run(150, graph_chunk=0)  # one sampling step short
    assert b.results()[0]["status"] == -1
    b.run(1, graph_chunk=0)
    assert b.results()[0]["status"] in (0, -5)


def test_long_window_groups_steps():
    # beyond 65,536 sampled steps each series entry is the mean of B steps
    # (B = 2 here, one step in front left out): 70,001 steps -> 35,000 entries
    ctx = hmd.Context(hmd.Params(n_equil=0, **SMALL_L))
    b = hmd.Batch(ctx, [(6.0, 0.05, 2, 70001)])
    b.run(70001, graph_chunk=100)
    q = b.series(0)
    assert len(q) == 35000
    assert np.all(q != 0.0)
    r = b.results()[0]
    assert r["status"] in (0, -5)
    assert r["flux"] == pytest.approx(q.mean(), rel=1e-12)
    assert r["flux_se"] == pytest.approx(ostats.geyer(q)[1], rel=1e-9)


@pytest.mark.parametrize("path", [1, 2, 3])
def test_pressure_series_from_identical_state(path):
    # Alg. 1's pressure output of a run: per sampled step the normal force of
    # the walls on the fluid per unit area, (F_lo,y - F_hi,y) / (2 Lx Lz).
    # From one equilibrated state both sides step 40 times; each step's
    # pressure agrees to FP32-force rounding (the first step exactly so up to
    # it), at a density other than the context's (the job's own)
    rho = 0.72
    pre = omd.System(7.0, 0.03, 9, omd.Params(rho=rho, **SMALL_L))
    pre.run(300)
    x, v = pre.get_state()
    n = 40
    params = dict(n_equil=0, **SMALL_L)
    ora = omd.System(7.0, 0.03, 9, omd.Params(rho=rho, cell_w=2.8, **params))
    ora.set_state(x, v)
    ora.run(n)
    po = ora.pressure_series()
    ctx = hmd.Context(hmd.Params(force_path=path, skin=0.3, pressure=1, **params))
    b = hmd.Batch(ctx, [(7.0, 0.03, 9, n, rho)])
    assert b.n_fluid(0) == ora.n_fluid
    b.set_state(0, x, v)
    b.run(n, graph_chunk=20)
    pg = b.pressure_series(0)
    assert len(pg) == n == len(po)
    assert np.abs(pg - po).max() <= 1e-4 * np.abs(po).mean(), np.abs(pg - po).max()
    assert abs(pg[0] - po[0]) <= 1e-5 * abs(po[0])
    r = b.results()[0]
    m, se = ostats.geyer(pg)
    assert r["p"] == pytest.approx(m, rel=1e-12) and r["p_se"] == pytest.approx(se, rel=1e-9)
    # the flux of the same run is unchanged by recording the pressure
    ctx0 = hmd.Context(hmd.Params(force_path=path, skin=0.3, **params))
    b0 = hmd.Batch(ctx0, [(7.0, 0.03, 9, n, rho)])
    b0.set_state(0, x, v)
    b0.run(n, graph_chunk=20)
    assert np.abs(b0.series(0) - b.series(0)).max() <= 1e-9 * np.abs(b.series(0)).max()
    assert b0.results()[0]["p"] == 0.0
    with pytest.raises(hmd.HmdError):
        b0.pressure_series(0)


def test_per_job_density_and_pressure_rejected_on_the_cell_path():
    # jobs at their own densities start from the oracle's lattice at that
    # density; the cell path does not record the wall pressure
    ctx = hmd.Context(hmd.Params(n_equil=0, **SMALL_L))
    jobs = [(6.0, 0.01, 3, 10, 0.65), (6.0, 0.01, 3, 10, 0.9), (6.0, 0.01, 3, 10)]
    b = hmd.Batch(ctx, jobs)
    for k, rho in enumerate((0.65, 0.9, 0.8)):
        o = omd.System(6.0, 0.01, 3, omd.Params(rho=rho, **SMALL_L))
        assert b.n_fluid(k) == o.n_fluid
        x, v = b.get_state(k)
        xo, vo = o.get_state()
        assert np.array_equal(x, xo) and np.abs(v - vo).max() <= 1e-14
    with pytest.raises(hmd.HmdError):
        hmd.Batch(hmd.Context(hmd.Params(force_path=0, pressure=1, **SMALL_L)), jobs[:1])


def test_full_batch_pressure_matches_oracle_wall_forces():
    # the 64-channel batch (2,115,470 atoms, default path and skin), each
    # channel at its own density around 0.8, with the wall pressure on and
    # sampling from the first step: the last sampled step's pressure of the
    # thinnest, a middle and the thickest channel equals the oracle's wall
    # normal force per area at that state, (F_lo,y - F_hi,y) / (2 Lx Lz)
    box = workloads.batch_box()
    params = dict(n_equil=0, **box)
    ctx = hmd.Context(hmd.Params(skin=0.35, pressure=1, **params))
    jobs = workloads.batch_jobs(64)
    rhos = [0.72 + 0.16 * (k % 5) / 4 for k in range(64)]
    n = 300
    b = hmd.Batch(ctx, [(j.h, j.g, j.seed, n, r) for j, r in zip(jobs, rhos)])
    b.run(n, graph_chunk=100)
    hs = [j.h for j in jobs]
    for sim in sorted({int(np.argmin(hs)), 31, int(np.argmax(hs))}):
        x, v = b.get_state(sim)
        ps = b.pressure_series(sim)
        assert len(ps) == n and np.all(np.isfinite(ps))
        j = jobs[sim]
        o = omd.System(j.h, j.g, j.seed, omd.Params(rho=rhos[sim], cell_w=2.5 + 0.35, **params))
        assert o.n_fluid == b.n_fluid(sim)
        o.set_state(x, v)
        fd = o.force_diag()
        po = 0.5 * (fd["wall_lo"][1] - fd["wall_hi"][1]) / (o.Lx * o.Lz)
        assert ps[-1] == pytest.approx(po, rel=1e-5), (sim, ps[-1], po)
    # every channel's result is the mean of its own per-step series, with a
    # finite, non-negative standard error (the first 300 steps from the
    # lattice are a transient: no sign is fixed for the pressure there)
    r = b.results()
    bad = []
    for k, q in enumerate(r):
        ps = b.pressure_series(k)
        if not (q["status"] in (0, -5) and q["p"] == pytest.approx(ps.mean(), rel=1e-12, abs=1e-12)
                and np.isfinite(q["p_se"]) and q["p_se"] >= 0.0):
            bad.append((k, q["status"], q["p"], ps.mean(), q["p_se"]))
    assert not bad, bad[:8]
