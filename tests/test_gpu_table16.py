"""The paper's 16-point tabulated-profile kappa (RT_KAPPA_TABLE16) through
the C ABI against the FP64 oracle: within 1e-5 relative, exact zeros where
the oracle is zero (the 16-point membership is integer work), every gas."""
from dataclasses import replace

import numpy as np
import pytest

from paper_cs_0703028_amd import inputs as I

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.fixture(scope="module")
def rt():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_cs_0703028_amd import rtlbl
    return rtlbl


@pytest.fixture(scope="module")
def O():
    from oracle import oracle
    return oracle


def _rel(g, o):
    nz = o != 0
    assert (g[~nz] == 0).all(), "GPU nonzero where the oracle is exactly zero"
    return np.abs(g[nz] - o[nz]) / np.abs(o[nz])


@pytest.mark.parametrize("wl", ["small_ragged", "plain_8cube", "small_ragged_two_gases"])
def test_table16_kappa_matches_oracle(rt, O, wl):
    w = getattr(I, wl)()
    t = rt.Tracer(0)
    t.setup_workload(w)
    print(f"table16 kappa {wl}", flush=True)
    kap, _ = t.compute_kappa(rt.KAPPA_TABLE16)
    n_nu = w.lines.n_nu
    kg = kap.cpu().numpy().astype(np.float64)
    ko = O.kappa_table16(w.grid, w.lines)
    for g in w.gases:
        ko = ko + O.kappa_table16(replace(w.grid, x=g.x), g.lines)
    assert (kg[:, n_nu:] == 0).all()
    r = _rel(kg[:, :n_nu], ko)
    print(f"  rel err max {r.max():.3e} median {np.median(r):.3e}", flush=True)
    assert r.max() <= REL
    st = t.stats()
    n_lines = len(w.lines.nu) + sum(len(g.lines.nu) for g in w.gases)
    assert st["line_evals"] <= 16 * n_lines * w.grid.n_cells
    t.close()


def test_table16_tallies_match_oracle_march(rt, O):
    w = I.plain_8cube()
    t = rt.Tracer(0)
    t.setup_workload(w)
    t.compute_kappa(rt.KAPPA_TABLE16)
    t.trace_rays(w.seed, w.n_rays, 0, w.n_rays, 0)
    ag, eg, _ = t.tally()
    g = w.grid
    Or, Dr, _ = O.rays(w.seed, 0, w.n_rays, g.nx, g.ny, g.nz)
    kap = O.kappa_table16(g, w.lines)
    a, e, _, _ = O.march(g, w.lines, Or, Dr, O.ray_weight(g, w.lines, w.n_rays), kap,
                         O.planck_rows(g, w.lines))
    ra, re = _rel(ag, a), _rel(eg, e)
    print(f"table16 tallies: absorbed max {ra.max():.3e}, emitted max {re.max():.3e}", flush=True)
    assert ra.max() <= REL and re.max() <= REL
    t.close()


def test_table16_needs_eight_point_cutoff(rt):
    w = I.small_ragged()
    t = rt.Tracer(0)
    t.setup_grid(w.grid)
    t.setup_lines(replace(w.lines, cutoff=5 * w.lines.dnu))
    with pytest.raises(rt.RtError) as e:
        t.compute_kappa(rt.KAPPA_TABLE16)
    assert e.value.status == rt.RT_EUNSUPPORTED
    t.close()


def test_table16_full_size_32cube_sampled_rows(rt, O):
    """The 16-point kappa of the whole 32^3 table (20,000 lines, 50,000
    points), as bench computes it; 64 seeded cells' rows against the oracle."""
    import torch
    w = I.plain_32cube()
    t = rt.Tracer(0)
    t.setup_workload(w)
    kap, _ = t.compute_kappa(rt.KAPPA_TABLE16)
    cells = np.sort(np.random.default_rng(12).choice(w.grid.n_cells, 64, replace=False))
    kg = kap[torch.as_tensor(cells, device=kap.device)].cpu().numpy().astype(np.float64)
    t.close()
    del kap
    torch.cuda.empty_cache()
    n_nu = w.lines.n_nu
    ko = O.kappa_table16(w.grid, w.lines, cells.astype(np.int32))
    assert (kg[:, n_nu:] == 0).all()
    r = _rel(kg[:, :n_nu], ko)
    print(f"table16 32^3 sampled rows: rel err max {r.max():.3e} median {np.median(r):.3e}",
          flush=True)
    assert r.max() <= REL


@pytest.mark.parametrize("cells,n_nu,n_lines,huge", [
    ((1, 1, 1), 1, 3, 0), ((7, 3, 3), 255, 40, 0), ((4, 4, 4), 256, 63, 0),
    ((5, 13, 1), 257, 64, 0), ((8, 8, 2), 545, 200, 0), ((3, 3, 3), 800, 900, 0),
    ((9, 5, 3), 1600, 0, 0), ((5, 13, 1), 700, 100, 3),
])
def test_table16_tile_edges(rt, O, cells, n_nu, n_lines, huge):
    """Grids around a tile's 64 cells, spectra around its 256 points and 32-point
    parts, staged runs of up to, at and beyond 64 lines.  huge: lines whose
    amplitude is beyond float reach their own 16 points and no others."""
    nx, ny, nz = cells
    g = I.linear_T_grid(nx, 0.1, ny=ny, nz=nz, x=0.2)
    L = I.line_list(n_lines, 999.9, 1000.1 + n_nu * 0.01, seed=n_nu, dnu=0.01, n_nu=n_nu)
    for k in range(huge):
        L.S[7 + 30 * k] = 1e300
    t = rt.Tracer(0)
    t.setup_grid(g)
    t.setup_lines(L)
    print(f"table16 edges {cells} {n_nu} points {n_lines} lines", flush=True)
    kap, _ = t.compute_kappa(rt.KAPPA_TABLE16)
    kg = kap.cpu().numpy().astype(np.float64)
    t.close()
    ko = O.kappa_table16(g, L)
    assert (kg[:, n_nu:] == 0).all()
    fits = ko < 1e30
    assert fits.all() == (huge == 0)
    assert not np.isfinite(kg[:, :n_nu][~fits]).any()
    r = _rel(np.where(fits, kg[:, :n_nu], 0), np.where(fits, ko, 0))
    assert r.size == 0 or r.max() <= REL


@pytest.mark.parametrize("cells,n_nu,n_lines,huge", [
    ((1, 1, 1), 1, (3, 2), 0), ((5, 13, 1), 257, (3, 200), 0), ((8, 8, 1), 256, (64, 1, 65), 0),
    ((7, 3, 3), 545, (0, 130, 0, 64), 0), ((5, 13, 1), 700, (100, 90), 2),
])
def test_table16_gases_share_one_launch(rt, O, cells, n_nu, n_lines, huge):
    """Two to four gases with lists from a few lines to several stages, some
    of zero strengths.  huge: lines of the last gas whose
    amplitude is beyond float."""
    nx, ny, nz = cells
    g = I.linear_T_grid(nx, 0.1, ny=ny, nz=nz, x=0.2)
    lists = [I.line_list(max(n, 1), 999.9, 1000.1 + n_nu * 0.01, seed=n_nu + k, dnu=0.01, n_nu=n_nu)
             for k, n in enumerate(n_lines)]
    for L, n in zip(lists, n_lines):
        if n == 0:  # a list whose lines absorb nothing
            L.S[:] = 0.0
    for k in range(huge):
        lists[-1].S[7 + 30 * k] = 1e300
    t = rt.Tracer(0)
    t.setup_grid(g)
    t.setup_lines(lists[0])
    gases = [I.Gas(np.full(g.n_cells, 0.05 * (k + 1)), L) for k, L in enumerate(lists[1:])]
    for k, gas in enumerate(gases, start=1):
        t.setup_gas(k, gas)
    print(f"table16 gases {cells} {n_nu} points {n_lines} lines", flush=True)
    kap, _ = t.compute_kappa(rt.KAPPA_TABLE16)
    kg = kap.cpu().numpy().astype(np.float64)
    t.close()
    ko = O.kappa_table16(g, lists[0])
    for gas in gases:
        ko = ko + O.kappa_table16(replace(g, x=gas.x), gas.lines)
    assert (kg[:, n_nu:] == 0).all()
    fits = ko < 1e30
    assert fits.all() == (huge == 0)
    assert not np.isfinite(kg[:, :n_nu][~fits]).any()
    r = _rel(np.where(fits, kg[:, :n_nu], 0), np.where(fits, ko, 0))
    assert r.size == 0 or r.max() <= REL
