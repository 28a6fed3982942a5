"""Tables of more blocks than one launch may hold (2^32 threads) go out in
several launches: the split that the line sums' launches use, compiled alone on
the host, over tables up to the card's memory and around the limit.  A batch of
more rays than its march launch may hold is refused before anything is launched.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIMIT = (1 << 32) - 1

PROGRAM = r"""
#include <cstdio>
#include "launch_pieces.h"
int main() {
  long long groups, per, extra, threads;
  while (std::scanf("%lld %lld %lld %lld", &groups, &per, &extra, &threads) == 4) {
    const bool ok = rt::for_pieces(groups, per, extra, threads,
        [](int64_t first, int64_t n, int64_t blocks, bool last) {
          std::printf("%lld %lld %lld %d ", (long long)first, (long long)n, (long long)blocks, last);
          return true;
        });
    std::printf("%d\n", ok);
  }
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("pieces")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_cs_0703028_amd", "csrc"), str(d / "p.cpp"), "-o",
                    str(d / "p")], check=True, capture_output=True)

    def run(groups, per, extra, threads):
        out = subprocess.run([str(d / "p")], input=f"{groups} {per} {extra} {threads}\n", check=True,
                             capture_output=True, text=True).stdout.split()
        v = [int(x) for x in out[:-1]]
        return [v[i:i + 4] for i in range(0, len(v), 4)], out[-1] == "1"

    return run


def _check(pieces, groups, per, extra, threads):
    at = 0
    for k, (first, n, blocks, last) in enumerate(pieces):
        assert first == at and n >= 1 and blocks == n * per
        assert last == (k == len(pieces) - 1)
        assert (blocks + (extra if last else 0)) * threads <= LIMIT
        at += n
    assert at == groups


# (cells, points, points of a block's tile, threads): half tiles and the adaptive
# sum (256 points), whole tiles (512), the precision form (512 points, 512 threads)
@pytest.mark.parametrize("cells,n_nu,tile,threads", [
    (64 ** 3, 140000, 256, 256), (64 ** 3, 140000, 512, 512), (96 ** 3, 50000, 256, 256),
    (96 ** 3, 50000, 512, 512), (96 ** 3, 50000, 512, 256), (100 ** 3, 68000, 256, 256),
    (32 ** 3, 50000, 256, 256), (5 * 6 * 7, 3037, 256, 256), (8, (1 << 24) - 1, 256, 256),
])
def test_tables_up_to_the_cards_memory(split, cells, n_nu, tile, threads):
    ld = -(-n_nu // 1536) * 1536
    groups, per, walls = -(-cells // 8), -(-ld // tile), ld // 256
    pieces, ok = split(groups, per, walls, threads)
    assert ok
    _check(pieces, groups, per, walls, threads)
    if (groups * per + walls) * threads <= LIMIT:
        assert len(pieces) == 1


@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("over", [-1, 0, 1])
@pytest.mark.parametrize("per,extra", [(1, 0), (1, 7), (3, 0), (1000, 600)])
def test_around_the_limit(split, threads, over, per, extra):
    groups = (LIMIT // threads - extra) // per + over
    pieces, ok = split(groups, per, extra, threads)
    assert ok and len(pieces) == (2 if over > 0 else 1)
    _check(pieces, groups, per, extra, threads)


def test_one_group_that_does_not_fit(split):
    assert split(4, LIMIT // 256 + 1, 0, 256) == ([], False)
    assert split(4, 1, LIMIT // 256, 256) == ([], False)
    assert split(0, 5, 0, 256) == ([], True)


LIB = os.path.join(ROOT, "paper_cs_0703028_amd", "librtlbl.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="librtlbl.so not built")
@pytest.mark.parametrize("n_rays,fits", [((1 << 26) - 32, True), (1 << 26, False), (1 << 30, False)])
def test_batch_rays(n_rays, fits):
    """On a host-only handle, which stops where the first device call would be;
    the workspace's size is answered for any number of rays."""
    import ctypes as C

    from paper_cs_0703028_amd import inputs as I
    from paper_cs_0703028_amd import rtlbl as rt
    L = I.line_list(5, 1000.0, 1001.0, seed=1, dnu=0.01, n_nu=100)
    case = I.Workload("c", I.linear_T_grid(2, 0.1), L, n_rays, 1)
    host = rt.Tracer.host_only()
    host.setup_lines(L)
    arr, keep = host._cases([case])
    tun = rt.Tracer.default_tuning()
    tun.mode, tun.slots = rt.BATCH_PERSISTENT, 2
    for t, want in ((None, rt.RT_EUNSUPPORTED if fits else rt.RT_EINVAL), (tun, rt.RT_EUNSUPPORTED)):
        size = host.batch_workspace_size([case], t)
        assert size > 0
        assert rt.lib.rt_batch_prepare(host._h, 1, arr, rt.KAPPA_PLAIN, C.byref(t) if t else None,
                                       C.c_void_p(256), size) == want
    host.close()
