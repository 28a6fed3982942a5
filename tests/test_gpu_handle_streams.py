"""A handle on a stream of its own, one that the null stream does not wait for:
its counters are cleared on that stream, and the whole path gives the bits of a
handle on the null stream.
"""
import numpy as np
import pytest

from paper_cs_0703028_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_new_handles_on_a_stream_of_their_own():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_cs_0703028_amd import rtlbl as rt
    w = I.small_ragged()
    side = torch.cuda.Stream()

    def run():
        t = rt.Tracer(0)
        t.setup_grid(w.grid)
        first = t.tally()  # before any ray: the first use of the cleared sums
        t.setup_lines(w.lines)
        t.compute_kappa(rt.KAPPA_PLAIN)
        t.trace_rays(w.seed, w.n_rays)
        out = t.tally()
        t.close()
        return first, out

    print("null stream", flush=True)
    _, ref = run()
    for k in range(3):
        print(f"own stream {k}", flush=True)
        with torch.cuda.stream(side):
            first, out = run()
        assert all((a == 0).all() for a in first)
        for a, b in zip(out, ref):
            assert np.array_equal(a, b)
