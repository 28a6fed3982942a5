"""The plain march where its forms meet: spectra that end at, before and after
its 768-point chunk and the 1536-point table pitch, the Planck cubics and the
general Planck values (wide point spacings), and gas from
transparent (the segment sums over a) to thick (the sums over t), per cell
against the FP64 oracle.  The tolerance is the repository's 1e-5 per cell.
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


def _run(rt, w):
    t = rt.Tracer(0)
    t.setup_workload(w)
    t.compute_kappa(rt.KAPPA_PLAIN)
    t.trace_rays(w.seed, w.n_rays, 0, w.n_rays, rt.TALLY_F32)
    out = t.tally()
    t.close()
    return out


def _check(got, ref):
    for g, o in zip(got, (ref["absorbed"], ref["emitted"], ref["balance"])):
        nz = o != 0
        assert (g[~nz] == 0).all()
        assert (np.abs(g[nz] - o[nz]) <= REL * np.abs(o[nz])).all()


@pytest.mark.parametrize("n_nu,dnu,x,T_wall", [
    (1, 0.01, 0.1, 900.0), (767, 0.01, 0.1, 0.0), (768, 0.01, 0.1, 900.0),
    (769, 0.01, 0.3, 0.0), (1535, 0.01, 1e-3, 900.0), (1537, 0.01, 1e-5, 900.0),
    (2304, 0.02, 1.0, 0.0), (1600, 0.05, 0.1, 900.0), (1600, 0.25, 1e-4, 900.0),
])
def test_chunk_ends_planck_forms_and_optical_depths(rt, O, n_nu, dnu, x, T_wall):
    g = I.linear_T_grid(4, 0.1, ny=3, nz=5, T_lo=300.0, T_hi=1800.0, x=x, p=1.1, T_wall=T_wall)
    L = I.line_list(300, 999.0, 1001.0 + n_nu * dnu, seed=4, dnu=dnu, n_nu=n_nu)
    w = I.Workload("edges", g, L, 300, 6)
    print(f"n_nu {n_nu} dnu {dnu} x {x}", flush=True)
    _check(_run(rt, w), O.run(g, L, w.n_rays, seed=w.seed))


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [12287, 12288, 12289, 20001])
def test_coherent_order_starts_at_12288_rays(rt, n, prec):
    """One call of n rays against pieces of it below the order's first batch
    size: the tallies are exact sums of the same values."""
    t = rt.Tracer(0)
    t.setup_workload(I.small_ragged())
    t.compute_kappa(rt.KAPPA_COMPENSATED)  # with the Planck table, which both forms take
    print(f"{n} rays, {prec}", flush=True)
    p = rt.TALLY_F64 if prec == "f64" else rt.TALLY_F32
    t.trace_rays(7, n, 0, n, p)
    one = t.tally()
    t.reset_tally()
    for b in range(0, n, 5000):
        t.trace_rays(7, n, b, min(5000, n - b), p)
    for a, b in zip(one, t.tally()):
        assert np.array_equal(a, b)
    t.close()


U = 1 << 21  # one cell width


@pytest.mark.parametrize("o,d", [
    ((0, 0, 0), (1, 1, 1)), ((0, 0, 0), (1, 1, 0)), ((0, 0, 0), (0, 1, 1)),
    ((0, 0, 0), (2, 1, 2)), ((0, U, 0), (1, 0, 1)), ((4 * U, 3 * U, 5 * U), (-1, -1, -1)),
    ((4 * U, U // 2, U), (-2, 1, 1)), ((0, U, 2 * U), (1, 0, 0)), ((U, 3 * U, 5 * U - 1), (0, -1, 0)),
    ((3 * U, 0, U), (-1, 1, 1)), ((1, 3 * U, 4 * U), (1, -1, -1)),
])
def test_rays_through_edges_and_corners(rt, O, o, d):
    """Rays that reach two or three planes at once, and rays along an axis or
    in a plane: every cell's power against the oracle's own traversal."""
    g = I.linear_T_grid(4, 0.1, ny=3, nz=5, T_lo=400.0, T_hi=1500.0, x=0.1, T_wall=900.0)
    L = I.line_list(200, 999.0, 1011.0, seed=3, dnu=0.01, n_nu=1000)
    o = np.array([o], np.int64)
    d = np.array([d], np.int64) << 19
    t = rt.Tracer(0)
    t.setup_grid(g)
    t.setup_lines(L)
    t.compute_kappa(rt.KAPPA_PLAIN)
    print(f"ray {o[0]} {d[0]}", flush=True)
    t.trace_explicit(o, d, 1.0)
    got = t.tally()
    t.close()
    a, e, b, _ = O.march(g, L, o, d, 1.0, O.kappa(g, L), O.planck_rows(g, L))
    _check(got, {"absorbed": a, "emitted": e, "balance": b})


def test_tally_grid_sizes_and_repeats(rt, O):
    """One handle over grids of one cell, around a block's 256 cells and around
    the 2^16 cells up to which results come through host memory: powers against
    the oracle, and a second tally the same bits."""
    t = rt.Tracer(0)
    for cells in [(1, 1, 1), (64, 2, 2), (257, 1, 1), (3, 4, 5), (256, 256, 1), (257, 256, 1), (5, 5, 5)]:
        g = I.linear_T_grid(cells[0], 0.02, ny=cells[1], nz=cells[2], T_lo=500.0, T_hi=1500.0, x=0.1,
                            T_wall=800.0)
        L = I.line_list(40, 999.9, 1001.1, seed=5, dnu=0.01, n_nu=100)
        print(f"tally {cells}", flush=True)
        t.setup_grid(g)
        t.setup_lines(L)
        t.compute_kappa(rt.KAPPA_PLAIN)
        t.trace_rays(3, 200)
        one = t.tally()
        for a, b in zip(one, t.tally()):
            assert np.array_equal(a, b)
        _check(one, O.run(g, L, 200, seed=3))
        t.reset_tally()
        assert all((a == 0).all() for a in t.tally())
    t.close()
