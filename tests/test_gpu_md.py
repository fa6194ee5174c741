"""Parity of the HIP NEMD path with the FP64 oracle, through the C ABI.

Bars: bit-exact initial state, cell membership and pair-list membership from
identical FP64 positions (pairs within 1e-5 relative of the list cut-off
excepted: FP32 and FP64 may legitimately disagree there); per-atom FP32
forces within 1e-5 relative RMS of the FP64 oracle; mass flux within the
combined standard error of independent runs.  Both force paths (cell list
every step, Verlet pair list) are checked.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

hmd = pytest.importorskip("paper_1603_04628_amd")
from oracle import md as omd  # noqa: E402
import workloads  # noqa: E402

SMALL_L = dict(Lx_nom=workloads.BOX_SMALL_LITERAL, Lz_nom=workloads.BOX_SMALL_LITERAL)
SMALL = dict(Lx_nom=workloads.BOX_SMALL, Lz_nom=workloads.BOX_SMALL, n_fluid=2048)
LARGE = dict(Lx_nom=workloads.BOX_LARGE, Lz_nom=workloads.BOX_LARGE)
SKIN = 0.3
PATHS = [0, 1, 2, 3]  # cell lists, pair lists, LDS-staged tiles, tiles on the gather fallback


def _pair(h, g, seed, path=1, **params):
    ctx = hmd.Context(hmd.Params(force_path=path, skin=SKIN, **params))
    cell_w = 2.5 + SKIN if path >= 1 else 0.0
    return ctx, hmd.System(ctx, h, g, seed), omd.System(h, g, seed, omd.Params(cell_w=cell_w, **params))


def _rel_rms(f, fo):
    return np.sqrt(((f.astype(np.float64) - fo) ** 2).sum() / (fo ** 2).sum())


def _per_atom_ok(f, fo):
    # atom by atom: FP32 rounding stays far below 1e-3 (eps/sigma); a pair
    # missing or extra anywhere inside the cut-off would add at least
    # |F(rc)| = 0.039.  Only pairs within FP32 rounding of the cut-off may
    # differ (reading of the membership rule), which moves a few atoms by at
    # most one pair force at rc.
    d = np.abs(f.astype(np.float64) - fo).max(axis=1)
    off = d > 1e-3
    return off.sum() <= 6 and (d[off] <= 0.045).all(), (int(off.sum()), float(d.max()))


@pytest.mark.parametrize("h,params", [(6.0, SMALL_L), (6.0, SMALL), (4.0, SMALL_L), (15.0, SMALL_L)])
def test_initial_state_is_identical(h, params):
    ctx, g_sys, o_sys = _pair(h, 0.02, 11, **params)
    assert (g_sys.n_fluid, g_sys.n_wall, g_sys.ncell) == (o_sys.n_fluid, o_sys.n_wall, o_sys.ncell)
    x, v = g_sys.get_state()
    xo, vo = o_sys.get_state()
    assert np.array_equal(x, xo)
    assert np.abs(v - vo).max() <= 1e-14


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("h,params,steps", [(6.0, SMALL_L, 300), (6.0, SMALL, 300), (4.0, SMALL_L, 100),
                                            (12.0, SMALL_L, 200)])
def test_cell_membership_bit_exact(h, params, steps, path):
    ctx, g_sys, o_sys = _pair(h, 0.02, 5, path, **params)
    assert g_sys.config()["path"] == min(path, 2)
    o_sys.run(steps)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    cell_g, cnt_g, order_g = g_sys.cells()
    cell_o, cnt_o, order_o = o_sys.cells()
    assert np.array_equal(cell_g.astype(np.int64), cell_o.astype(np.int64))
    assert np.array_equal(cnt_g.astype(np.int64), cnt_o.astype(np.int64))
    start = np.concatenate([[0], np.cumsum(cnt_o)[:-1]])
    for c in range(len(cnt_o)):
        a = np.sort(order_g[start[c]:start[c] + cnt_o[c]].astype(np.int64))
        b = np.sort(order_o[start[c]:start[c] + cnt_o[c]].astype(np.int64))
        assert np.array_equal(a, b)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("h", [14.3, 17.0, 29.0, 100.0])
def test_sort_of_many_cells(h, path):
    # 2,000 to 14,000 cells of a dilute channel: the scan of a system's cells in
    # one round of 2,048, in two with a part left, in several; slots in cell
    # order, every cell complete
    params = dict(rho=0.05, **LARGE)
    ctx, g_sys, o_sys = _pair(h, 0.02, 5, path, **params)
    o_sys.run(100)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    (cell_g, cnt_g, order_g), (cell_o, cnt_o, _) = g_sys.cells(), o_sys.cells()
    assert np.array_equal(cell_g.astype(np.int64), cell_o.astype(np.int64))
    assert np.array_equal(cnt_g.astype(np.int64), cnt_o.astype(np.int64))
    by_cell = cell_o.astype(np.int64)[order_g.astype(np.int64)]
    assert np.all(np.diff(by_cell) >= 0)
    assert np.array_equal(np.sort(order_g.astype(np.int64)), np.arange(o_sys.n_fluid))


@pytest.mark.parametrize("path", PATHS)
def test_cell_sort_is_stable(path):
    # the counting sort keeps the previous slot order inside every cell:
    # sorting an already sorted state changes nothing, and after the atoms
    # move, the members of a new cell that came from one old cell keep
    # their old relative order (bit-exact, whatever the cell numbering)
    ctx, g_sys, o_sys = _pair(6.0, 0.02, 9, path, **SMALL_L)
    o_sys.run(100)
    x1, v1 = o_sys.get_state()
    g_sys.set_state(x1, v1)
    cell1, cnt1, order1 = (a.astype(np.int64) for a in g_sys.cells())
    g_sys.set_state(x1, v1)
    _, _, order2 = (a.astype(np.int64) for a in g_sys.cells())
    assert np.array_equal(order2, order1)
    o_sys.run(40)
    x3, v3 = o_sys.get_state()
    g_sys.set_state(x3, v3)
    cell3, cnt3, order3 = (a.astype(np.int64) for a in g_sys.cells())
    assert np.any(cell3 != cell1)  # some atoms changed cells
    rank1 = np.empty_like(order1)
    rank1[order1] = np.arange(len(order1))  # position of each atom in the old order
    start3 = np.concatenate([[0], np.cumsum(cnt3)[:-1]])
    for c in np.nonzero(cnt3)[0]:
        m = order3[start3[c]:start3[c] + cnt3[c]]
        assert np.all(cell3[m] == c)
        for oc in np.unique(cell1[m]):
            sub = m[cell1[m] == oc]
            assert np.all(np.diff(rank1[sub]) > 0), (c, oc)


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("n_in", [40, 56, 57, 100])
def test_sort_of_crowded_cells(n_in, path):
    # a cell up to, at and past its bucket (56 entries here): members complete
    # and in their old order, every other cell too
    ctx, g_sys, o_sys = _pair(6.0, 0.02, 9, path, **SMALL_L)
    x, v = g_sys.get_state()
    cell1, _, order1 = (a.astype(np.int64) for a in g_sys.cells())
    rank1 = np.empty_like(order1)
    rank1[order1] = np.arange(len(order1))
    inside = np.all((x > 0.05) & (x < 2.7), axis=1)
    x[inside] += 2.9  # out of the first cell
    pick = np.random.default_rng(n_in).choice(len(x), n_in, replace=False)
    grid = np.stack(np.meshgrid(*[np.arange(5) * 0.5 + 0.3] * 3, indexing="ij"), -1).reshape(-1, 3)
    x[pick] = grid[:n_in]
    g_sys.set_state(x, v)
    cell, cnt, order = (a.astype(np.int64) for a in g_sys.cells())
    assert np.array_equal(np.bincount(cell, minlength=len(cnt)), cnt)
    assert cnt[cell[pick[0]]] >= n_in and np.all(cell[pick] == cell[pick[0]])
    start = np.concatenate([[0], np.cumsum(cnt)[:-1]])
    for c in np.nonzero(cnt)[0]:  # cells are reported row by row, not in slot order: one old cell at a time
        m = order[start[c]:start[c] + cnt[c]]
        assert np.array_equal(np.sort(m), np.nonzero(cell == c)[0])
        for oc in np.unique(cell1[m]):
            assert np.all(np.diff(rank1[m[cell1[m] == oc]]) > 0), (c, oc)


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("n_fluid,n_in", [(200, 32), (200, 33), (200, 55), (200, 56), (200, 57), (200, 90), (0, 72),
                                          (0, 73)])
def test_sort_of_cells_at_their_bucket(n_fluid, n_in, path):
    # 30 sigma^3 cells: buckets of 56 entries in a vapour of 6 atoms per cell
    # (room for condensed fluid; twice the mean and some would be 32), of 72 in
    # the liquid.  A cell up to, at and past them: members complete and in
    # their old order, every other cell too
    ctx, g_sys, o_sys = _pair(6.0, 0.02, 9, path, n_fluid=n_fluid, **SMALL_L)
    x, v = g_sys.get_state()
    cell1, _, order1 = (a.astype(np.int64) for a in g_sys.cells())
    rank1 = np.empty_like(order1)
    rank1[order1] = np.arange(len(order1))
    corner = np.all(x < np.array([o_sys.Lx / 4, 3.0, o_sys.Lz / 4]) + 1e-6, axis=1)
    x[corner, 0] += 0.3 * o_sys.Lx
    pick = np.random.default_rng(n_in).choice(len(x), n_in, replace=False)
    grid = np.stack(np.meshgrid(*[np.arange(5) * 0.5 + 0.3] * 3, indexing="ij"), -1).reshape(-1, 3)
    x[pick] = grid[:n_in]
    g_sys.set_state(x, v)
    cell, cnt, order = (a.astype(np.int64) for a in g_sys.cells())
    assert np.array_equal(np.bincount(cell, minlength=len(cnt)), cnt)
    assert cnt[cell[pick[0]]] == n_in and np.all(cell[pick] == cell[pick[0]])
    start = np.concatenate([[0], np.cumsum(cnt)[:-1]])
    for c in np.nonzero(cnt)[0]:
        m = order[start[c]:start[c] + cnt[c]]
        assert np.array_equal(np.sort(m), np.nonzero(cell == c)[0])
        for oc in np.unique(cell1[m]):
            assert np.all(np.diff(rank1[m[cell1[m] == oc]]) > 0), (c, oc)


@pytest.mark.parametrize("h,skin,cell_w,params", [
    (3.0, 0.3, 0.0, SMALL_L),  # one cell between the walls: every range of a column
    (5.0, 0.25, 0.0, LARGE),   # thin and wide: columns on both sides of an origin block
    (6.0, 0.3, 4.0, SMALL_L),  # three slabs and columns: tiles over the whole row, partial last groups
    (9.0, 0.3, 6.0, SMALL),    # wide cells: ranges of more than one part
    (8.0, 0.9, 0.0, SMALL),    # long lists: more entries than an atom's LDS row holds
    (20.0, 0.35, 0.0, SMALL),  # tall columns
    (60.0, 0.3, 0.2, SMALL_L)])
def test_tiled_list_build_shapes(h, skin, cell_w, params):
    # forces from lists screened on the matrix cores, against the oracle's
    # forces: FP32 pair forces reach 1e-6 relative RMS, a lost pair in reach
    # would show as a single-atom error (as _per_atom_ok)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=skin, cell_w=cell_w, **params))
    g_sys, o_sys = hmd.System(ctx, h, 0.02, 8), omd.System(h, 0.02, 8, omd.Params(**params))
    o_sys.run(60)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    f, pe = g_sys.forces()
    fo, peo = o_sys.forces_cells()
    ok, info = _per_atom_ok(f, fo)
    assert ok, info
    assert pe == pytest.approx(peo, rel=1e-4)


@pytest.mark.parametrize("h", [24.0, 26.0, 30.0, 36.0])
def test_tall_channels(h):
    # columns whose neighbourhoods hold about 2,300, 2,470, 2,770 and 3,200
    # atoms: either LDS capacity and beyond both; bounds as above
    params = dict(Lx_nom=12.7, Lz_nom=12.7)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=0.3, **params))
    g_sys, o_sys = hmd.System(ctx, h, 0.02, 9), omd.System(h, 0.02, 9, omd.Params(**params))
    o_sys.run(40)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    f, pe = g_sys.forces()
    fo, peo = o_sys.forces_cells()
    ok, info = _per_atom_ok(f, fo)
    assert ok, info
    assert pe == pytest.approx(peo, rel=1e-4)
    o_sys.run(20)
    g_sys.run(20)
    d = g_sys.get_state()[0] - o_sys.get_state()[0]
    d -= o_sys.Lx * np.round(d / o_sys.Lx) * np.array([1, 0, 1])
    assert np.abs(d).max() <= 1e-3


@pytest.mark.parametrize("h,cell_w", [(4.0, 0.0), (9.0, 0.0), (15.0, 0.0), (4.0, 4.0), (8.0, 4.0), (12.0, 4.0),
                                      (19.0, 4.0), (21.0, 4.0), (24.0, 4.0)])
def test_lists_shared_by_lanes(h, cell_w):
    # columns of about 25 to 170 atoms (eight to one lanes per list) and 260 to
    # 340 (a second pass of few), with padded (four slabs) and partial (three
    # slabs) last groups; bounds as above
    params = dict(Lx_nom=12.7, Lz_nom=12.7)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=0.3, cell_w=cell_w, **params))
    g_sys, o_sys = hmd.System(ctx, h, 0.02, 9), omd.System(h, 0.02, 9, omd.Params(**params))
    o_sys.run(60)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    f, pe = g_sys.forces()
    fo, peo = o_sys.forces_cells()
    ok, info = _per_atom_ok(f, fo)
    assert ok, info
    assert pe == pytest.approx(peo, rel=1e-4)


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("heights,pressure", [((6.0,), 0), ((4.0, 9.0, 15.0), 0), ((4.0, 9.0), 1)])
def test_joined_launches_match_separate_ones(heights, pressure, path):
    # a step's sort, lists and forces in joined launches, against the separate
    # launches of timed steps: 60 steps with several rebuilds from one state.
    # The same FP32 pair forces up to the rounding of fused multiply-adds
    # (1e-7), which 60 steps of 0.005 amplify to well below 1e-4
    out = []
    for timed in (False, True):
        ctx = hmd.Context(hmd.Params(force_path=path, skin=SKIN, pressure=pressure, n_equil=20, **SMALL_L))
        b = hmd.Batch(ctx, [(h, 0.02, 7, 40) for h in heights])
        b.set_timing(timed)
        b.run(60, graph_chunk=20 if not timed else 0)
        out.append([b.get_state(k)[0] for k in range(len(heights))] + [b.series(k) for k in range(len(heights))])
        if timed:
            assert b.kernel_ms("scan")[1] == 60
    n = len(heights)
    for k in range(n):
        d = out[0][k] - out[1][k]
        L = omd.System(heights[k], 0.02, 7, omd.Params(**SMALL_L)).Lx
        d -= L * np.round(d / L)
        assert np.abs(d).max() <= 1e-4, k
        np.testing.assert_allclose(out[0][n + k], out[1][n + k], rtol=0, atol=1e-4)


def _tile_shapes(b, o, x):
    """Per tile of a one-channel batch (or of equal channels), from the host's
    geometry: staged atoms, home atoms, entries of the longest run of three
    columns' fluid; and cells of a tile's neighbourhood."""
    nx, ny, nz = o.ncell
    ntx = b.tuning()["tiles"] // (nz * b.n)
    L = np.array([o.Lx, o.Lz])

    def columns(p):
        c = np.minimum((p[:, [0, 2]] / L * [nx, nz]).astype(int), [nx - 1, nz - 1])
        return np.bincount(c[:, 1] * nx + c[:, 0], minlength=nx * nz).reshape(nz, nx)

    fluid, both = columns(x), columns(np.vstack([x, o.wall()]))
    staged, home = [], []
    for z in range(nz):
        zs = sorted({(z - 1) % nz, z, (z + 1) % nz})
        for t in range(ntx):
            x0, x1 = t * nx // ntx, (t + 1) * nx // ntx
            xs = sorted({c % nx for c in range(x0 - 1, x1 + 1)})
            staged.append(both[np.ix_(zs, xs)].sum())
            home.append(fluid[z, x0:x1].sum())
    runs = fluid + np.roll(fluid, 1, 1) + np.roll(fluid, -1, 1)
    cells = 3 * min(-(-nx // ntx) + 2, nx) * (ny + 2)
    return dict(staged=max(staged), home=(min(home), max(home)), run=runs.max(), cells=cells, ny=ny)


def _forces_of_one(b, k, h, seed, params, cell_w=0.0):
    """Forces of channel k of a batch and its state against the oracle; returns
    the oracle's system and the state."""
    x, v = b.get_state(k)
    f, pe = b.forces(k)
    o = omd.System(h, 0.02, seed, omd.Params(cell_w=max(2.5 + SKIN, cell_w), **params))
    o.set_state(x, v)
    fo, peo = o.forces_cells()
    ok, info = _per_atom_ok(f, fo)
    assert ok, info
    assert pe == pytest.approx(peo, rel=1e-4)
    return o, x


@pytest.mark.parametrize("h,n_fluid,ny,table,stage", [
    (179.0, 2000, 63, True, 0),      # cells across: one lane each in the lookup
    (179.4, 2000, 64, True, 0),
    (182.1, 2000, 65, True, 0),      # two
    (233.0, 2000, 83, True, 0),      # the last the table holds
    (236.0, 2000, 84, False, 0),     # cell by cell, staged in LDS
    (300.0, 2000, 107, False, 0),
    (300.0, 3500, 107, False, 1)])   # past TILE_STAGE: cell by cell, from memory
def test_list_build_of_dilute_tall_channels(h, n_fluid, ny, table, stage):
    # forces from the lists as in test_tiled_list_build_shapes; the tile's
    # neighbourhood fits the force kernels' LDS, which side of the cell table it
    # lies on is asserted from the geometry
    params = dict(Lx_nom=12.7, Lz_nom=12.7, n_fluid=n_fluid)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=SKIN, **params))
    b = hmd.Batch(ctx, [(h, 0.02, 8, 0)])
    b.run(60, graph_chunk=20)
    o, x = _forces_of_one(b, 0, h, 8, params)
    s = _tile_shapes(b, o, x)
    assert s["ny"] == ny and (s["cells"] <= 768) == table, s
    assert (2400 < s["staged"] < 3072) if stage else s["staged"] < 2400, s


@pytest.mark.parametrize("n_in", [255, 256, 290])
def test_list_build_of_a_crowded_cell(n_in):
    # a cell of up to 255 atoms is in the table's range, more are not: its
    # neighbours' tiles build cell by cell, within the LDS capacity
    params = dict(n_fluid=500, wall_layers=1, Lx_nom=workloads.BOX_SMALL, Lz_nom=workloads.BOX_SMALL)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=SKIN, cell_w=6.0, **params))
    b = hmd.Batch(ctx, [(13.0, 0.02, 8, 0)])
    x, v = b.get_state(0)
    o = omd.System(13.0, 0.02, 8, omd.Params(cell_w=6.0, **params))
    grid = np.stack(np.meshgrid(*[np.arange(7) * 0.95 + 0.45] * 3, indexing="ij"), -1).reshape(-1, 3)
    grid[:, 1] += 0.5
    grid = grid[np.all(grid < np.array([o.Lx / 3, 6.5, o.Lz / 3]), axis=1)][:n_in]
    rest = x[(x[:, 0] > 8.0) & (x[:, 0] < o.Lx - 0.6)][:500 - n_in]
    xs = np.vstack([grid, rest])
    assert xs.shape == x.shape
    b.set_state(0, xs, v)
    o, x = _forces_of_one(b, 0, 13.0, 8, params, cell_w=6.0)
    cell, cnt, _ = o.cells()
    assert cnt.max() == n_in
    s = _tile_shapes(b, o, x)
    assert s["staged"] < 2400 and s["cells"] <= 768, s


@pytest.mark.parametrize("n,h,cell_w,params,home,run,stage", [
    (6, 10.0, 0.0, LARGE, 257, 129, 2400),                          # second passes of up to 32 atoms
    (1, 34.0, 0.0, dict(Lx_nom=12.7, Lz_nom=12.7, wall_layers=1), 257, 129, 3072),
    (1, 37.2, 0.0, dict(Lx_nom=12.7, Lz_nom=12.7, wall_layers=1), 289, 129, 3072),  # of up to 64
    (1, 39.5, 0.0, dict(Lx_nom=12.7, Lz_nom=12.7, wall_layers=1), 321, 129, 3072),  # of up to 128
    (1, 8.0, 0.0, LARGE, 1, 129, 2400),                             # fluid ranges of two parts
    (1, 8.0, 4.0, LARGE, 1, 257, 2400)])                            # of three
def test_lds_tiles_of_many_atoms(n, h, cell_w, params, home, run, stage):
    # lists of LDS indices: tiles of more atoms than the workgroup has threads,
    # candidate ranges longer than the part screened at once.  That the tiles
    # keep within the LDS capacity and reach these branches is asserted from
    # the geometry
    ctx = hmd.Context(hmd.Params(force_path=2, skin=SKIN, cell_w=cell_w, **params))
    b = hmd.Batch(ctx, [(h, 0.02, 8, 0)] * n)
    b.run(60, graph_chunk=20)
    o, x = _forces_of_one(b, n - 1, h, 8, params, cell_w)
    s = _tile_shapes(b, o, x)
    assert s["home"][1] >= home and s["run"] >= run and s["staged"] < stage, s
    print(s)


@pytest.mark.parametrize("heights", [(6.0, 30.0), (6.0, 36.0), (6.0, 30.0, 36.0)])
def test_tall_channels_among_others(heights):
    # one capacity per batch: the larger for neighbourhoods of 2,770 atoms, the
    # smaller where 3,200 exceed both and gather from memory
    params = dict(Lx_nom=12.7, Lz_nom=12.7)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=SKIN, **params))
    b = hmd.Batch(ctx, [(h, 0.02, 9, 0) for h in heights])
    b.run(60, graph_chunk=20)
    for k, h in enumerate(heights):
        _forces_of_one(b, k, h, 9, params)


def test_lists_past_2_to_the_24_slots():
    # 16.8 M atoms: list groups lie beyond 4 GiB and a slot count beyond 24
    # bits.  The last channel's forces after 20 steps against the oracle's, bar
    # of test_forces_match_oracle_paper_scale_channel
    n = 429
    ctx = hmd.Context(hmd.Params(force_path=2, skin=SKIN, **LARGE))
    b = hmd.Batch(ctx, [(15.0, 0.02, 4, 0)] * n)
    print("created", b.atoms, flush=True)
    assert b.atoms > 2 ** 24
    b.run(20, graph_chunk=0)
    assert b.config()["path"] == 2
    x, v = b.get_state(n - 1)
    f, _ = b.forces(n - 1)
    o = omd.System(15.0, 0.02, 4, omd.Params(**LARGE))
    o.set_state(x, v)
    fo, _ = o.forces_cells()
    assert _rel_rms(f, fo) <= 1e-5
    ok, info = _per_atom_ok(f, fo)
    assert ok, info


@pytest.mark.parametrize("path", PATHS)
def test_pair_counts(path):
    # ordered fluid pairs and wall pairs inside the cut-off, counted directly;
    # a pair within FP32 rounding of it (1e-6 of the ~1e5 pairs) may go either way
    ctx = hmd.Context(hmd.Params(force_path=path, skin=SKIN, **SMALL_L))
    b = hmd.Batch(ctx, [(6.0, 0.02, 3, 0), (4.0, 0.02, 4, 0)])
    b.run(40, graph_chunk=20)
    ff, wf = b.pair_count()
    want = [0, 0]
    for k, h in enumerate((6.0, 4.0)):
        o = omd.System(h, 0.02, 3 + k, omd.Params(**SMALL_L))
        x, xw = b.get_state(k)[0], o.wall()
        for q, y in enumerate((x, xw)):
            for xi in x:
                d = y - xi
                for a, L in ((0, o.Lx), (2, o.Lz)):
                    d[:, a] -= L * np.round(d[:, a] / L)
                want[q] += int(np.sum(np.sum(d * d, axis=1) < 6.25)) - (1 if q == 0 else 0)
    assert abs(ff - want[0]) <= 4 and abs(wf - want[1]) <= 4, (ff, wf, want)


@pytest.mark.parametrize("path", [1, 2, 3])
@pytest.mark.parametrize("h,params,steps", [(6.0, SMALL_L, 300), (4.0, SMALL_L, 100), (12.0, SMALL_L, 200),
                                            (15.0, SMALL, 200)])
def test_pair_lists_match_oracle_neighbour_sets(h, params, steps, path):
    ctx, g_sys, o_sys = _pair(h, 0.02, 6, path, **params)
    o_sys.run(steps)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    rl = 2.5 + SKIN
    nb_g = g_sys.neighbors()
    nb_o = o_sys.neighbors(rl)
    xw = o_sys.wall()
    allx = np.vstack([xo, xw])
    Lx, Lz = o_sys.Lx, o_sys.Lz
    nmis = 0
    for i in range(o_sys.n_fluid):
        a, b = set(nb_g[i].tolist()), set(nb_o[i].tolist())
        for j in a ^ b:  # disagreements only at the cut-off, within FP32 rounding
            d = xo[i] - allx[j]
            d[0] -= Lx * np.round(d[0] / Lx)
            d[2] -= Lz * np.round(d[2] / Lz)
            assert abs(d @ d - rl * rl) <= 1e-5 * rl * rl, (i, j, d @ d)
            nmis += 1
    assert nmis <= 2


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("h,params,steps", [(6.0, SMALL_L, 500), (6.0, SMALL, 500), (4.0, SMALL_L, 200),
                                            (15.0, SMALL_L, 300)])
def test_forces_match_oracle(h, params, steps, path):
    ctx, g_sys, o_sys = _pair(h, 0.03, 2, path, **params)
    o_sys.run(steps)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    f, pe = g_sys.forces()
    fo, peo = o_sys.forces_cells()
    assert _rel_rms(f, fo) <= 1e-5
    ok, info = _per_atom_ok(f, fo)
    assert ok, info
    assert pe == pytest.approx(peo, rel=1e-5)


@pytest.mark.parametrize("path", PATHS)
def test_forces_match_oracle_paper_scale_channel(path):
    # 39,189 atoms at h = 15 in the 57 x 57 box, from the start lattice
    ctx, g_sys, o_sys = _pair(15.0, 0.02, 0, path, **LARGE)
    assert g_sys.n_fluid == 39189
    f, pe = g_sys.forces()
    fo, peo = o_sys.forces_cells()
    assert _rel_rms(f, fo) <= 1e-5
    o_sys.run(20)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    f, _ = g_sys.forces()
    fo, _ = o_sys.forces_cells()
    assert _rel_rms(f, fo) <= 1e-5
    ok, info = _per_atom_ok(f, fo)
    assert ok, info


@pytest.mark.parametrize("path", PATHS)
def test_short_trajectory_tracks_oracle(path):
    ctx, g_sys, o_sys = _pair(6.0, 0.05, 3, path, **SMALL_L)
    o_sys.run(200)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    o_sys.run(40)
    g_sys.run(40)
    xg, vg = g_sys.get_state()
    xo, vo = o_sys.get_state()
    d = xg - xo
    d[:, 0] -= g_sys.Lx * np.round(d[:, 0] / g_sys.Lx)
    d[:, 2] -= g_sys.Lz * np.round(d[:, 2] / g_sys.Lz)
    assert np.sqrt((d ** 2).mean()) < 1e-5
    assert np.sqrt(((vg - vo) ** 2).mean()) < 1e-4


@pytest.mark.parametrize("path", PATHS)
def test_nve_energy_fluctuation_matches_oracle(path):
    ctx, g_sys, o_sys = _pair(6.0, 0.0, 1, path, **SMALL_L)
    o_sys.run(1000)
    xo, vo = o_sys.get_state()
    g_sys.set_state(xo, vo)
    o_sys.set_state(xo, vo)
    eg = g_sys.run(400, thermostat=False, energy=True)
    eo = o_sys.run(400, thermostat=False, energy=True)
    assert abs(eg[0] - eo[0]) < 1e-5 * abs(eo[0])
    assert eg.std() == pytest.approx(eo.std(), rel=0.15)
    assert abs(eg[-1] - eg[0]) < 5e-4


def test_thermostat_holds_target():
    p = hmd.Params(n_equil=500, **SMALL_L)
    ctx = hmd.Context(p)
    r = hmd.md_flux_batch(ctx, [(6.0, 0.0, 4, 2000)])[0]
    assert r["status"] == 0
    assert r["T"][1] == pytest.approx(1.0, abs=0.01)


FLUX_PARAMS = dict(n_equil=3000, rho=0.6, **SMALL_L)
FLUX_SEEDS = list(range(7, 19))


@pytest.fixture(scope="module")
def oracle_flux():
    return [omd.md_flux(6.0, 0.1, s, 8000, omd.Params(**FLUX_PARAMS)) for s in FLUX_SEEDS]


@pytest.mark.parametrize("path", PATHS)
def test_flux_matches_oracle_within_standard_errors(path, oracle_flux):
    # liquid channel (rho = 0.6 over the wall gap), one independent run per
    # seed on each side, on every force path; the error of each mean is the
    # spread over seeds.  A check across the paths: four comparisons at once,
    # so |t| <= 3.5 keeps the family's false-alarm rate near 1% (22 degrees
    # of freedom).  The 2-standard-error bar on the benchmark's own channels
    # is test_gpu_flux_parity.py.
    ctx = hmd.Context(hmd.Params(force_path=path, **FLUX_PARAMS))
    gres = hmd.md_flux_batch(ctx, [(6.0, 0.1, s, 8000) for s in FLUX_SEEDS])
    dg = np.array([r["flux"] for r in gres])
    do = np.array([r["flux"] for r in oracle_flux])
    n = len(FLUX_SEEDS)
    t = (dg.mean() - do.mean()) / np.sqrt(dg.var(ddof=1) / n + do.var(ddof=1) / n)
    print("flux gpu", dg, "oracle", do, "t", t)
    assert all(r["status"] == 0 for r in gres)
    assert abs(t) <= 3.5  # two-sided p < 0.003 per path
    # temperatures are reported with the step's Berendsen factor applied
    for r, o in zip(gres, oracle_flux):
        assert r["T"][1] == pytest.approx(o["T"][1], abs=0.01)


@pytest.mark.parametrize("path", PATHS)
def test_profile_bins_match_oracle(path):
    # Sec. 2.1: every sampled step also adds each atom's streamwise velocity
    # and a count to the wall-normal bin of its height.  From one equilibrated
    # state, ten sampled steps on each side differ only by FP32 force rounding:
    # the counts agree exactly and the momentum sums far below one velocity.
    pre = omd.System(6.0, 0.05, 7, omd.Params(**SMALL_L))
    pre.run(300)
    x, v = pre.get_state()
    ctx, g_sys, o_sys = _pair(6.0, 0.05, 7, path, n_equil=0, **SMALL_L)
    g_sys.set_state(x, v)
    o_sys.set_state(x, v)
    g_sys.run(10)
    o_sys.run(10)
    mvx, cnt = g_sys.profile()
    mvo, cno = o_sys.profile()
    assert cno.sum() == 10 * o_sys.n_fluid
    assert np.array_equal(cnt, cno)
    assert np.abs(mvx - mvo).max() <= 1e-6 * max(1.0, np.abs(mvo).max())


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("bins", [150, 208, 209, 240])
def test_profiles_of_many_bins_match_oracle(bins, path):
    # a workgroup holds 208 bins; those past them are added to atom by atom; bars
    # of test_profile_bins_match_oracle
    fine = dict(SMALL_L, bin_dy=6.0 / (bins - 0.5))
    pre = omd.System(6.0, 0.05, 7, omd.Params(**fine))
    pre.run(300)
    x, v = pre.get_state()
    ctx, g_sys, o_sys = _pair(6.0, 0.05, 7, path, n_equil=0, **fine)
    g_sys.set_state(x, v)
    o_sys.set_state(x, v)
    g_sys.run(10)
    o_sys.run(10)
    mvx, cnt = g_sys.profile()
    mvo, cno = o_sys.profile()
    assert len(cnt) == len(cno) == bins
    assert np.array_equal(cnt, cno)
    assert np.abs(mvx - mvo).max() <= 1e-6 * max(1.0, np.abs(mvo).max())


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("S", [1, 16, 17])
def test_temperatures_of_a_batch_are_those_of_its_states(S, path):
    # thermostat and temperature sums start cache lines of their own, 16 sums
    # to a line.  Rounding of sums of a thousand terms, in another order.
    ctx = hmd.Context(hmd.Params(force_path=path, **SMALL_L))
    b = hmd.Batch(ctx, [(4.0 + 0.25 * k, 0.02, 3 + k, 4) for k in range(S)])
    want = np.zeros((S, 3))
    for _ in range(4):
        b.run(1, 0)
        want += [(b.get_state(k)[1] ** 2).mean(axis=0) for k in range(S)]
    for r, w in zip(b.results(), want):
        np.testing.assert_allclose(r["T"], w / 4.0, rtol=1e-12)


@pytest.mark.parametrize("S,h,rho", [(17, 12.0, 0.2), (16, 12.0, 0.2), (1, 16.0, 0.4)])
def test_tiles_of_fluids_below_a_liquids_density(S, h, rho):
    # 17 such channels have more than 1,280 tiles and take the larger LDS capacity,
    # 16 do not; and one whose tiles keep room for denser places.  Bars of the
    # other force tests.
    p = dict(LARGE, rho=rho)
    ctx = hmd.Context(hmd.Params(force_path=2, skin=SKIN, **p))
    b = hmd.Batch(ctx, [(h, 0.01, 3 + k, 10) for k in range(S)])
    b.run(100, 50)
    k = S - 1
    x, v = b.get_state(k)
    o = omd.System(h, 0.01, 3 + k, omd.Params(cell_w=2.5 + SKIN, **p))
    o.set_state(x, v)
    f, fo = b.forces(k)[0], o.forces_cells()[0]
    assert _rel_rms(f, fo) <= 1e-5
    ok, worst = _per_atom_ok(f, fo)
    assert ok, worst


def test_batch_equals_single_systems():
    p = hmd.Params(**SMALL_L)
    ctx = hmd.Context(p)
    jobs = [(4.5, 0.01, 1, 0), (7.0, 0.02, 2, 0), (11.0, 0.03, 3, 0)]
    b = hmd.Batch(ctx, jobs)
    assert b.atoms == sum(hmd.System(ctx, h, g, s).n_fluid for h, g, s, _ in jobs)
    b.run(50, graph_chunk=10)
    res = b.results()
    for (h, g, s, _), r in zip(jobs, res):
        single = hmd.Batch(ctx, [(h, g, s, 0)])
        single.run(50, graph_chunk=0)
        r1 = single.results()[0]
        assert r1["pe"] == pytest.approx(r["pe"], rel=1e-3)


def test_downloads_of_batches_that_share_a_context():
    # the context's pinned buffer serves every batch of it and grows with the
    # largest download: small and large in turn, after the small one is freed
    # too, as from contexts of their own
    small, large = (dict(h=5.0, n=40), dict(h=15.0, n=9000))
    own = []
    for c in (small, large):
        b = hmd.Batch(hmd.Context(hmd.Params(**SMALL_L)), [(c["h"], 0.02, 3, c["n"])])
        b.run(20, graph_chunk=0)
        own.append((b.get_state(0), b.series(0), b.results()))
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    bs = [hmd.Batch(ctx, [(c["h"], 0.02, 3, c["n"])]) for c in (small, large)]
    for b in bs:
        b.run(20, graph_chunk=0)
    for k in (0, 1, 0, 1):
        if bs[k] is None:
            continue
        (x, v), q, r = own[k]
        xs, vs = bs[k].get_state(0)
        assert np.abs(xs - x).max() <= 1e-6 and np.abs(vs - v).max() <= 1e-4
        assert np.abs(bs[k].series(0) - q).max() <= 1e-4
        assert bs[k].results()[0]["pe"] == pytest.approx(r[0]["pe"], rel=1e-5)
        if k == 0:
            bs[0].close()
            bs[0] = None


@pytest.mark.parametrize("path", PATHS)
def test_graph_replay_equals_direct_launches(path):
    # same steps as direct launches and as graph replays: trajectories agree
    # to FP32 force rounding (reductions run in a different order)
    ctx = hmd.Context(hmd.Params(force_path=path, **SMALL_L))
    a = hmd.System(ctx, 6.0, 0.02, 9)
    b = hmd.Batch(ctx, [(6.0, 0.02, 9, 0)])
    a.run(40)  # shorter than the default graph chunk: direct launches
    b.run(40, graph_chunk=20)
    pe_a = a.forces()[1] / a.n_fluid
    assert b.results()[0]["pe"] == pytest.approx(pe_a, rel=1e-4)


def test_paths_agree_on_a_trajectory():
    out = []
    for path in PATHS:
        ctx = hmd.Context(hmd.Params(force_path=path, **SMALL_L))
        s = hmd.System(ctx, 6.0, 0.05, 12)
        s.run(60)
        out.append(s.get_state())
    for other in out[1:]:
        d = out[0][0] - other[0]
        d[:, 0] -= s.Lx * np.round(d[:, 0] / s.Lx)
        d[:, 2] -= s.Lz * np.round(d[:, 2] / s.Lz)
        assert np.sqrt((d ** 2).mean()) < 1e-4


def test_unstable_system_is_reported():
    # two atoms 0.05 sigma apart blow up within a few steps: the run's
    # result carries HMD_EUNSTABLE
    p = hmd.Params(n_equil=0, **SMALL_L)
    ctx = hmd.Context(p)
    b = hmd.Batch(ctx, [(6.0, 0.0, 0, 4)])
    x, v = b.get_state(0)
    x[1] = x[0] + [0.05, 0.0, 0.0]
    b.set_state(0, x, v)
    b.run(4, graph_chunk=0)
    r = b.results()[0]
    assert r["status"] == hmd.binding.HMD_EUNSTABLE
    xg, vg = b.get_state(0)
    assert not np.all(np.isfinite(vg)) or np.abs(vg).max() > 1e3


def test_invalid_arguments_are_rejected():
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    with pytest.raises(hmd.HmdError):
        hmd.System(ctx, 1.0, 0.0, 0)  # h below twice the start gap
    with pytest.raises(hmd.HmdError):
        hmd.md_flux_batch(ctx, [(6.0, 0.0, 0, 1)])  # one sample has no standard error
    with pytest.raises(hmd.HmdError):
        hmd.System(hmd.Context(hmd.Params(thermo_axis=0, **SMALL_L)), 6.0, 0.0, 0)  # thermostat on the flow


def test_autotuner_picks_a_configuration():
    # coordinate descent over path, skin (0.05 steps), tile size, cell width
    # and graph chunk; the fastest candidate is what a later batch of the
    # same workload uses, and its results match an untuned run's physics
    ctx = hmd.Context(hmd.Params(**SMALL_L))
    jobs = [(6.0, 0.02, k, 0) for k in range(4)]
    table = hmd.binding.md_autotune(ctx, jobs, probe_steps=40)
    cols = hmd.binding.TUNE_COLUMNS
    assert table.shape[1] == len(cols) and len(table) >= 10 and np.all(table[:, 6] > 0)
    assert {0, 1, 2} <= set(table[:, 0].astype(int).tolist())
    assert {0.25, 0.30, 0.40, 0.45} <= set(np.round(table[table[:, 0] >= 1, 1], 2).tolist())
    b = hmd.Batch(ctx, jobs)
    best = table[np.argmin(table[:, 6])]
    tun = b.tuning()
    assert tun["path"] == int(best[0]) and tun["tpb"] == int(best[2])
    assert tun["graph_chunk"] == int(best[5])
    if best[0] >= 1:
        assert tun["skin"] == pytest.approx(best[1])
    assert tun["tile_alpha"] == pytest.approx(best[3])
    assert tun["cell_width"] >= 2.5


def test_full_batch_forces_match_oracle():
    # the 64-channel batch as the benchmark runs it (2,115,470 atoms, default
    # path and skin, graph chunks of 100): after 300 steps, the forces of the
    # thinnest, a middle and the thickest system at their device state match
    # the oracle's from the same positions
    params = dict(n_equil=10000, **workloads.batch_box())
    ctx = hmd.Context(hmd.Params(skin=0.35, **params))
    jobs = workloads.batch_jobs(64)
    b = hmd.Batch(ctx, [(j.h, j.g, j.seed, 20000) for j in jobs])
    assert b.atoms == 2115470
    b.run(300, graph_chunk=100)
    hs = [j.h for j in jobs]
    for sim in sorted({int(np.argmin(hs)), 31, int(np.argmax(hs))}):
        x, v = b.get_state(sim)
        f, pe = b.forces(sim)
        j = jobs[sim]
        o = omd.System(j.h, j.g, j.seed, omd.Params(cell_w=2.5 + 0.35, **params))
        o.set_state(x, v)
        fo, peo = o.forces_cells()
        assert np.all(np.isfinite(f))
        assert _rel_rms(f, fo) <= 1e-5, sim
        ok, info = _per_atom_ok(f, fo)
        assert ok, (sim, info)
        assert pe == pytest.approx(peo, rel=1e-5)


def test_full_batch_sampled_outputs_hold_invariants():
    # the 64-channel batch (2,115,470 atoms, default path and skin) through
    # md_flux_batch with the benchmark's protocol (10k + 20k steps; a shorter
    # one leaves the widest channels' start-up flow unsettled, which the
    # library rightly reports as not stationary): every channel finishes, the
    # thermostatted component holds T0, the flux follows the body force
    # (never significantly against it, clearly with it where g h^3 is
    # largest), and J is the flux per unit height
    params = dict(n_equil=10000, **workloads.batch_box())
    ctx = hmd.Context(hmd.Params(skin=0.35, **params))
    jobs = workloads.batch_jobs(64)
    res = hmd.md_flux_batch(ctx, [(j.h, j.g, j.seed, 20000) for j in jobs])
    assert sum(r["n_fluid"] for r in res) == 2115470
    drive = np.array([j.g * j.h ** 3 for j in jobs])
    strong = set(np.argsort(drive)[-16:].tolist())
    for k, (j, r) in enumerate(zip(jobs, res)):
        assert r["status"] == 0, k
        assert r["T"][1] == pytest.approx(1.0, abs=0.02), k
        assert np.isfinite(r["flux"]) and r["flux_se"] > 0.0, k
        assert r["flux"] > -4.0 * r["flux_se"], k
        if k in strong:
            assert r["flux"] > 3.0 * r["flux_se"], k
        assert r["jflux"] == pytest.approx(r["flux"] / j.h, rel=1e-12), k


def test_timed_graph_replays_report_kernel_times():
    # with timing on, one graph replay in ten stamps the device clock around
    # the kernels of ten of its steps (the others replay the plain graph):
    # every kernel gets a positive time and their sum stays within the
    # stamped replay's time per step
    params = dict(n_equil=10000, **workloads.batch_box())
    ctx = hmd.Context(hmd.Params(skin=0.35, **params))
    jobs = workloads.batch_jobs(8)
    b = hmd.Batch(ctx, [(j.h, j.g, j.seed, 20000) for j in jobs])
    b.run(20, graph_chunk=20)
    b.set_timing(True)
    b.run(400, graph_chunk=20)  # 20 replays: the 1st and 11th stamped
    step_ms, nsteps = b.kernel_ms("graph_step")
    assert nsteps == 40 and step_ms > 0.0
    total = 0.0
    for k in ("integrate", "keys", "scan", "scatter", "reorder", "list", "force"):
        ms, n = b.kernel_ms(k)
        assert n == 20 and ms > 0.0, k
        total += ms
    assert total <= 1.05 * step_ms
    assert b.kernel_ms("force")[0] > 0.2 * step_ms
    # the list build apart on stamped steps that rebuild and that do not
    (tr, nr), (ti, ni) = b.kernel_ms("list_rebuild"), b.kernel_ms("list_idle")
    assert nr + ni == 20 and ni > 0
    if nr > 0:
        assert tr > 5.0 * ti
        assert (nr * tr + ni * ti) / 20 == pytest.approx(b.kernel_ms("list")[0], rel=1e-9)


@pytest.mark.parametrize("h,rho,box", [(6.0, 0.8, SMALL_L), (4.2, 0.8, LARGE), (9.87, 0.72, SMALL_L),
                                       (15.0, 0.9, SMALL_L)])
def test_initial_state_meets_the_reading(h, rho, box):
    # the library's start lattice against the reading itself, not the
    # oracle: N_f = round(rho Lx Lz h) atoms on planes within [delta, h -
    # delta] (delta = 1), no two closer than the lattice allows, velocities
    # with zero mean and exactly T0 over 3 N_f degrees of freedom, drawn
    # normal (kurtosis 3) before the rescale
    ctx = hmd.Context(hmd.Params(n_equil=0, **box))
    b = hmd.Batch(ctx, [(h, 0.01, 21, 10, rho)])
    x, v = b.get_state(0)
    n = b.n_fluid(0)
    o = omd.System(h, 0.01, 21, omd.Params(rho=rho, **box))  # only for the snapped box extents
    Lx, Lz = o.Lx, o.Lz
    assert n == round(rho * Lx * Lz * h) == len(x)
    assert x[:, 1].min() >= 1.0 - 1e-12 and x[:, 1].max() <= h - 1.0 + 1e-12
    assert np.all((x[:, 0] >= 0) & (x[:, 0] < Lx) & (x[:, 2] >= 0) & (x[:, 2] < Lz))
    # plane structure: equally spaced planes from delta to h - delta
    ys = np.unique(np.round(x[:, 1], 9))
    if len(ys) > 1:
        assert ys[0] == pytest.approx(1.0, abs=1e-9) and ys[-1] == pytest.approx(h - 1.0, abs=1e-9)
        assert np.allclose(np.diff(ys), np.diff(ys)[0], rtol=1e-9)
    if n <= 5000:
        d = x[:, None, :] - x[None, :, :]
        d[..., 0] -= Lx * np.round(d[..., 0] / Lx)
        d[..., 2] -= Lz * np.round(d[..., 2] / Lz)
        r = np.sqrt((d ** 2).sum(-1))[np.triu_indices(n, 1)]
        assert r.min() > 0.95
    assert np.abs(v.mean(0)).max() < 1e-13
    assert (v ** 2).sum() / (3 * n) == pytest.approx(1.0, abs=1e-12)
    assert abs(np.mean(v ** 4) / np.mean(v ** 2) ** 2 - 3.0) < 0.5
