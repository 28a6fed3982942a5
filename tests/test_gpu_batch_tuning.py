"""A batch runs with the tuning that the caller gives; only where none is given
may the default's one slab run as two of half the points, in the same workspace
and to the same bits.  What a tuning runs as shows in the workspace, which holds
the slabs and one wall row per case, rounded up to whole chunks.
"""
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


def _cases(n_nu):
    L = I.line_list(60, 1000.0, 1000.0 + n_nu * 0.01, seed=2, dnu=0.01, n_nu=n_nu)
    return [I.Workload("c%d" % k, I.linear_T_grid(18, 0.05, x=0.1, T_wall=700.0), L, 3000, 5 + k)
            for k in range(3)]


def _tuning(rt, points, slots):
    t = rt.Tracer.default_tuning()
    t.chunk_points, t.slots = points, slots
    return t


@pytest.mark.parametrize("n_nu", [3072, 3073, 4608, 4609, 9300])
def test_workspace_of_the_given_tuning(rt, n_nu):
    t = rt.Tracer(0)
    cases = _cases(n_nu)
    t.setup_lines(cases[0].lines)
    C = rt.MARCH_CHUNK
    rows = lambda points: len(cases) * -(-n_nu // points) * points * 4
    slab = lambda points: sum(c.grid.n_cells for c in cases) * points * 4
    one, small = (t.batch_workspace_size(cases, _tuning(rt, p, 1)) for p in (2 * C, C))
    two = t.batch_workspace_size(cases, _tuning(rt, C, 2))
    up = 3 * 256  # each array's end is rounded up
    assert abs(one - small - (rows(2 * C) - rows(C)) - (slab(2 * C) - slab(C))) <= up
    assert abs(two - small - slab(C)) <= up
    # no tuning: the workspace of the default one, whichever way it runs
    assert t.batch_workspace_size(cases) == one
    assert t.batch_workspace_size(cases, rt.Tracer.default_tuning()) == one
    t.close()


@pytest.mark.parametrize("n_nu", [3072, 3073, 4700])
def test_no_tuning_and_one_slab_give_the_same_bits(rt, n_nu):
    """Prepared with no tuning (in halves beyond 3072 points) and with the
    default one given, each in the other's workspace."""
    cases = _cases(n_nu)
    t = rt.Tracer(0)
    t.setup_lines(cases[0].lines)
    print(f"no tuning, n_nu {n_nu}", flush=True)
    ws = t.batch_prepare(cases, rt.KAPPA_PLAIN)
    t.batch_launch()
    free = t.batch_results()
    t.batch_prepare(cases, rt.KAPPA_PLAIN, rt.Tracer.default_tuning(), ws)
    t.batch_launch()
    given = t.batch_results()
    t.close()
    for a, b in zip(free, given):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)


def test_a_tuning_timed_on_other_kernels_is_not_served(rt, tmp_path):
    """Entries of the cache's key v6 were timed on other line sums and marches,
    and some ran in halves unasked: they are timed anew."""
    import torch
    cases = [I.Workload("c", I.linear_T_grid(4, 0.1, x=0.1), I.line_list(
        20, 1000.0, 1010.0, seed=1, dnu=0.01, n_nu=1000), 100, 3)]
    t = rt.Tracer(0)
    t.setup_lines(cases[0].lines)
    big = _tuning(rt, 4 * rt.MARCH_CHUNK, 8)
    ws = torch.empty(t.batch_workspace_size(cases, big), dtype=torch.uint8, device="cuda")
    path = tmp_path / "tune.json"
    print("cache key", flush=True)
    t.batch_autotune(cases, rt.KAPPA_PLAIN, ws, str(path))
    text = path.read_text()
    key = text.split('"')[1]
    path.write_text('{\n  "v6|%s": [%d, 16, 64, 2, 7, 0]\n}\n'
                    % (key.split("|", 1)[1], 64 * rt.MARCH_CHUNK))
    best = t.batch_autotune(cases, rt.KAPPA_PLAIN, ws, str(path))
    assert best.chunk_points <= 4 * rt.MARCH_CHUNK and best.slots != 7
    assert key in path.read_text()
    t.close()
