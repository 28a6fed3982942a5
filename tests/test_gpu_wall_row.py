"""The walls' row is written in the plain line sum's launch, or in the Planck
table's where the caller asks for that: the same tallies bit for bit either way,
for half and whole tiles of the line sum, ragged spectra, and after
the walls' temperature changes on the same handle.
"""
from dataclasses import replace

import numpy as np
import pytest

from paper_cs_0703028_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_cs_0703028_amd import rtlbl
    return rtlbl


def _tallies(rt, t, grid, planck):
    t.setup_grid(grid)
    k, p = t.alloc_tables()
    t.compute_kappa(rt.KAPPA_PLAIN, k, p if planck else None)
    t.reset_tally()
    t.trace_rays(3, 500)
    return t.tally()


@pytest.mark.parametrize("nx,ny,nz,n_nu", [(3, 3, 3, 1), (3, 1, 3, 257), (5, 6, 7, 3037), (24, 24, 24, 1537)])
def test_the_same_row_from_either_launch(rt, nx, ny, nz, n_nu):
    print(f"{nx} x {ny} x {nz} cells, {n_nu} points", flush=True)
    g = I.linear_T_grid(nx, 0.05, ny=ny, nz=nz, T_lo=400.0, T_hi=1500.0, x=0.1)
    L = I.line_list(100, 990.0, 1010.0 + 0.01 * n_nu, seed=1, n_nu=n_nu)
    t = rt.Tracer(0)
    t.setup_grid(g)
    t.setup_lines(L)
    entering = []
    for T_wall in (900.0, 0.0, 1200.0):
        grid = replace(g, T_wall=T_wall)
        a, b = (_tallies(rt, t, grid, planck) for planck in (False, True))
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
        entering.append(a[2][0])
    assert entering[1] == 0.0 < entering[0] < entering[2]
    t.close()


@pytest.mark.parametrize("mode", ["COMPENSATED", "TABLE16", "ADAPTIVE", "ADAPTIVE_WINGS"])
@pytest.mark.parametrize("nx,ny,nz,n_nu", [(3, 1, 3, 1), (5, 6, 7, 1537)])
def test_every_form_writes_the_row(rt, mode, nx, ny, nz, n_nu):
    """Forms whose own launch writes the row, against the Planck table's launch."""
    print(f"{mode} {nx} x {ny} x {nz} cells, {n_nu} points", flush=True)
    g = I.linear_T_grid(nx, 0.05, ny=ny, nz=nz, T_lo=400.0, T_hi=1500.0, x=0.1)
    t = rt.Tracer(0)
    t.setup_grid(g)
    t.setup_lines(I.line_list(100, 990.0, 1010.0 + 0.01 * n_nu, seed=1, n_nu=n_nu))
    t.set_line_tolerance(1e-3)  # for the adaptive forms
    for T_wall in (900.0, 0.0, 1200.0):
        out = []
        for planck in (False, True):
            t.setup_grid(replace(g, T_wall=T_wall))
            k, p = t.alloc_tables()
            t.compute_kappa(getattr(rt, "KAPPA_" + mode), k, p if planck else None)
            t.reset_tally()
            t.trace_rays(3, 500)
            out.append(t.tally())
        for x, y in zip(*out):
            assert np.array_equal(x, y)
        assert (out[0][2][0] > 0.0) == (T_wall > 0.0)
    t.close()
