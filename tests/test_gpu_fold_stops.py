"""Folded scalar steps where right-hand sides stop while the launch that finds it
is still starting workgroups: as many as the device holds at once, and more."""
import pytest

from gpu_util import setup, to_gpu
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(outer=3, max_outer=500, check_every=8), dict(use_ras=0, inner_tol=0.1)])
@pytest.mark.parametrize("n", [1, 5])
def test_every_solve_ends_alike(kw, n):
    """The same right-hand sides ten times: the same iterations and bitwise the same
    solutions, each with a true residual below the tolerance."""
    dims = (16, 16, 16, 32)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 1002, None)
    b = synth.gaussian_spinor(dims, 93, n)
    for k in range(1, n, 2):   # others stop elsewhere
        b[k] = 0.0
        b[k, 100 * k, 1, 2] = 1.0
    g = to_gpu(b if n > 1 else b.reshape(-1, 4, 3))
    first = None
    for _ in range(10):
        x, info, rc = lat.solve(g, tol=1e-10, **kw)
        info = info if n > 1 else [info]
        assert rc == 0
        r = (lat.apply(x) - g).reshape(n, -1)
        assert bool((r.norm(dim=1) <= 1e-10 * g.reshape(n, -1).norm(dim=1)).all())
        got = [(i["outer_iters"], i["inner_iters_total"]) for i in info]
        if first is None:
            first = (x, got)
            print(kw, n, got, flush=True)
        assert got == first[1] and bool((x == first[0]).all())
