"""The plain line sum's far nodes: lines at both ends of the nodes' reach of a
span and of a pair of spans, windows from narrower than a span to wider than
the default, spectra that end at the edges of spans, pairs and tiles, and both
tile sizes of the launch.  Kappa against the FP64 oracle within the
repository's 1e-5 per point, with zeros exactly where the oracle has them.
"""
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
    oracle.build()
    return oracle


def _kappa(rt, grid, lines):
    t = rt.Tracer(0)
    t.setup_grid(grid)
    t.setup_lines(lines)
    k, _ = t.alloc_tables()
    t.compute_kappa(rt.KAPPA_PLAIN, k, None)
    out = k.cpu().numpy()
    t.close()
    return out


def _check(got, want, n_nu):
    assert (got[:, n_nu:] == 0).all()
    g = got[:, :n_nu].astype(np.float64)
    nz = want != 0
    assert (g[~nz] == 0).all()
    assert (np.abs(g[nz] - want[nz]) <= REL * want[nz]).all()


def _grid(n=9):
    g = I.linear_T_grid(n, 0.1, ny=1, nz=1, T_lo=300.0, T_hi=1700.0, x=0.1, p=1.2)
    return g


@pytest.mark.parametrize("K", [20, 63, 64, 130, 500, 1100])
@pytest.mark.parametrize("n_nu", [1, 63, 65, 128, 511, 1025])
def test_random_lines_windows_and_lengths(rt, O, K, n_nu):
    dnu = 0.01
    L = I.line_list(120, 1000.0 - K * dnu, 1000.0 + (n_nu + K) * dnu, seed=K + n_nu, dnu=dnu,
                    n_nu=n_nu, cutoff=K * dnu)
    print(f"K {K} n_nu {n_nu}", flush=True)
    g = _grid()
    _check(_kappa(rt, g, L), O.kappa(g, L), n_nu)


@pytest.mark.parametrize("at", [-236, -170, -109, -108, -107, -55, -54, -53, 0, 63, 115, 116, 117,
                                180, 233, 234, 235, 400])
@pytest.mark.parametrize("phi", [0.0, 0.999])
def test_one_line_at_the_ends_of_the_reach(rt, O, at, phi):
    """One line whose centre lies `at` points from a span's first point (span
    4, the first of a pair): every point of every span it reaches."""
    n_nu, dnu = 1300, 0.01
    nu = np.array([1000.0 + (256 + at + phi) * dnu])
    L = I.Lines(nu=nu, S=np.array([1e-20]), gamma=np.array([0.06]), n_T=np.array([0.5]),
                E_lower=np.array([400.0]), T_ref=I.T_REF, cutoff=5.0, nu0=1000.0, dnu=dnu,
                n_nu=n_nu)
    print(f"at {at} phi {phi}", flush=True)
    g = _grid(3)
    _check(_kappa(rt, g, L), O.kappa(g, L), n_nu)


def test_tile_sizes_give_the_same_values(rt):
    """The same cells in a launch of few blocks (256-point tiles) and of many
    (512-point tiles): the same rows bit for bit."""
    L = I.line_list(4000, 1000.0, 1100.0, seed=2, n_nu=10000)
    small = I.hot_spot_grid(4, seed=1)
    big = I.hot_spot_grid(16, seed=1)
    for a in ("T", "x", "p"):
        getattr(big, a)[:64] = getattr(small, a)
    ks, kb = _kappa(rt, small, L), _kappa(rt, big, L)
    assert np.array_equal(ks, kb[:64])


@pytest.mark.parametrize("K,lines,cells", [(256, 300, 1600), (257, 300, 1600), (500, 2000, 1600),
                                           (513, 2100, 1600), (500, 300, 1360), (500, 300, 1366)])
def test_whole_and_half_tiles(rt, O, K, lines, cells):
    """Launches at either side of each line between whole and half tiles (window,
    lines per point, blocks): sampled cells against the oracle."""
    n_nu, dnu = 1000, 0.01
    L = I.line_list(lines, 1000.0 - K * dnu, 1000.0 + (n_nu + K) * dnu, seed=K, dnu=dnu, n_nu=n_nu,
                    cutoff=K * dnu)
    g = I.linear_T_grid(cells, 0.1, ny=3, nz=1, T_lo=300.0, T_hi=1700.0, x=0.1)
    print(f"K {K} {lines} lines {g.n_cells} cells", flush=True)
    pick = np.arange(0, g.n_cells, 97, dtype=np.int32)
    _check(_kappa(rt, g, L)[pick], O.kappa(g, L, pick), n_nu)
