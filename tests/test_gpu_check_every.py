"""opts.check_every bounds the first queue of every inner solve."""
import pytest

from gpu_util import setup, to_gpu
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner_tol,max_outer,every", [(0.12, 2, 1), (0.12, 2, 2), (0.1, 3, 1)])
def test_short_queues_leave_nothing_idle(inner_tol, max_outer, every):
    """Inner solves of different lengths (16 or 26 iterations in 4 or 6 of them):
    queues that start at one or two iterations and then follow the observed rate end
    where each solve does, so no hop is launched after it; with a first queue as
    long as the solve before, 20 are."""
    from paper_1612_06556_amd import wcl
    dims = (8, 8, 8, 8)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 1001, None)
    b = to_gpu(synth.gaussian_spinor(dims, 63))
    wcl.wcl_profile(lat.h, 1)
    _, info, _ = lat.solve(b, raise_on_error=False, tol=1e-10, inner_tol=inner_tol, use_ras=0, max_outer=max_outer,
                           check_every=every)
    k = wcl.wcl_profile_read(lat.h, wcl.K_HOP)
    wcl.wcl_profile(lat.h, 0)
    print(info["inner_iters_total"], k["launches"], k["idle_launches"], flush=True)
    assert info["outer_iters"] == max_outer and info["inner_iters_total"] >= 2 * max_outer
    assert k["idle_launches"] == 0
