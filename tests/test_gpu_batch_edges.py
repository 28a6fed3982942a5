"""The batched launch where its paths meet: compensated sums over windows
narrower and wider than a span's reach, spectra that end in a span, and a
single slab that runs as two halves (enough cells, points and rays) against one
that does not.  Per cell against the FP64 oracle within the repository's 1e-5,
and bit for bit between launch shapes.
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


def _run(rt, cases, mode, tun):
    t = rt.Tracer(0)
    t.setup_lines(cases[0].lines)
    ws = t.batch_prepare(cases, mode, tun)
    t.batch_launch()
    out = t.batch_results()
    t.close()
    del ws
    return out


@pytest.mark.parametrize("K,n_nu", [(20, 257), (130, 1600), (500, 1025), (1100, 300)])
def test_compensated_windows(rt, O, K, n_nu):
    dnu = 0.01
    L = I.line_list(150, 1000.0 - K * dnu, 1000.0 + (n_nu + K) * dnu, seed=K, dnu=dnu, n_nu=n_nu,
                    cutoff=K * dnu)
    cases = [I.Workload("a", I.linear_T_grid(5, 0.1, ny=3, nz=1, x=0.1, T_wall=900.0), L, 200, 3),
             I.Workload("b", I.linear_T_grid(4, 0.05, x=0.2, p=1.3), L, 300, 4)]
    outs = []
    for shape in (rt.BATCH_CHUNKED, rt.BATCH_PERSISTENT):
        tun = rt.Tracer.default_tuning()
        tun.mode, tun.slots, tun.chunk_points = shape, 2, rt.MARCH_CHUNK
        print(f"compensated batch K {K} n_nu {n_nu} shape {shape}", flush=True)
        outs.append(_run(rt, cases, rt.KAPPA_COMPENSATED, tun))
    for w, got, other in zip(cases, *outs):
        ref = O.run(w.grid, L, w.n_rays, seed=w.seed)
        for g, h, o in zip(got, other, (ref["absorbed"], ref["emitted"], ref["balance"])):
            assert np.array_equal(g, h)
            nz = o != 0
            assert (g[~nz] == 0).all()
            assert (np.abs(g[nz] - o[nz]) <= REL * np.abs(o[nz])).all()


@pytest.mark.parametrize("n_nu", [3072, 3073, 4700])
def test_one_slab_in_halves(rt, n_nu):
    """18^3 cells: one slab of 3072 points (in halves beyond 3072 points), one of
    1536 and two of 1536 give the same bits."""
    L = I.line_list(60, 1000.0, 1000.0 + n_nu * 0.01, seed=2, dnu=0.01, n_nu=n_nu)
    cases = [I.Workload("c", I.linear_T_grid(18, 0.05, x=0.1, T_wall=700.0), L, 3000, 5)]
    outs = []
    for points, slots in ((2 * rt.MARCH_CHUNK, 1), (rt.MARCH_CHUNK, 1), (rt.MARCH_CHUNK, 2)):
        tun = rt.Tracer.default_tuning()
        tun.chunk_points, tun.slots = points, slots
        print(f"halves n_nu {n_nu} {points}/{slots}", flush=True)
        outs.append(_run(rt, cases, rt.KAPPA_PLAIN, tun)[0])
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert np.array_equal(a, b)
