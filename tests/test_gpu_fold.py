"""BiCGStab with the scalar steps folded into the vector updates (up to 1024
partial sums a term) and as launches of their own (more): right-hand sides
that stop at different iterations, at once (zero) and by breakdown."""
import numpy as np
import pytest

import oracle
from gpu_util import rel, require_gpu, setup, to_gpu, to_host
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu


_refs = {}


def _reference(orc, b, key):
    if key not in _refs:
        _refs[key] = orc.bicgstab_eo(b, 1e-13, 20000)[0]
    return _refs[key]


# half-sites / block: 2048 / 256 = 8 partials; 1024 (the last folded); 1040 (the first that is not)
@pytest.mark.parametrize("dims,block", [((8, 8, 8, 8), 256), ((16, 16, 16, 32), 64), ((20, 16, 16, 26), 64)])
@pytest.mark.parametrize("kw", [dict(outer=3, max_outer=2000), dict(use_ras=0, inner_tol=0.1),
                                dict(use_ras=0, inner_tol=0.1, inner_prec=16, inner_vec_prec=16, use_graph=1)])
def test_solves_either_side_of_the_fold(dims, block, kw):
    """x within 1e-8 of the oracle's 1e-13 solution, true residual <= 1e-10; the
    zero right-hand side returns zero, and each is what it is alone (1e-9: the
    vector updates of a batch add their sums over other workgroups)."""
    from paper_1612_06556_amd import wcl
    lat, orc, _ = setup(dims, -1, 0.115, 1.0, 61, None)
    wcl.wcl_set_tuning(lat.h, block, 2, 1, 0)
    b = synth.gaussian_spinor(dims, 62, 3)
    b[1] = 0.0
    b[2] = 0.0
    b[2, 5, 1, 2] = 1.0
    x, info, rc = lat.solve(to_gpu(b), tol=1e-10, **kw)
    assert rc == 0 and all(i["status"] == 0 for i in info)
    x = to_host(x)
    assert not x[1].any()
    for k in (0, 2):
        ref = _reference(orc, b[k], (dims, k))
        assert np.linalg.norm(b[k] - orc.D(x[k])) <= 1e-10 * np.linalg.norm(b[k])
        assert rel(x[k], ref) <= 1e-8
        one, _, _ = lat.solve(to_gpu(b[k]), tol=1e-10, **kw)
        print(dims, block, kw, k, info[k]["outer_iters"], info[k]["inner_iters_total"], rel(to_host(one), x[k]), flush=True)
        assert rel(to_host(one), x[k]) <= 1e-9
    wcl.wcl_set_tuning(lat.h, 256, 2, 1, 0)


def test_iteration_limits_inside_a_chunk():
    """max_outer not a multiple of the queue length: the iterate and count are
    those of that many iterations, however the checks fall."""
    from paper_1612_06556_amd import wcl
    dims = (8, 8, 8, 8)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 1001, None)
    b = to_gpu(synth.gaussian_spinor(dims, 63))
    for limit in (1, 3, 7):
        got = []
        for every in (1, 2, 5, 8):
            x, info, rc = lat.solve(b, raise_on_error=False, tol=1e-12, outer=wcl.OUTER_PLAIN64_EO, max_outer=limit,
                                    check_every=every)
            assert rc == wcl.WCL_ENOCONV and info["outer_iters"] == limit
            got.append(to_host(x))
        assert all(np.array_equal(g, got[0]) for g in got)


# half-sites 192 (part of a block), 1800 (eighth block part full), 138240 (past 512 blocks)
@pytest.mark.parametrize("dims", [(4, 4, 4, 6), (6, 10, 6, 10), (24, 24, 24, 20)])
@pytest.mark.parametrize("kw", [dict(use_ras=0), dict(), dict(use_ras=0, inner_prec=16, inner_vec_prec=16)])
def test_a_solve_starts_from_nothing_left_over(dims, kw):
    """The search vectors of an earlier solve do not reach the next: bitwise what
    a new lattice gives, and a true residual within the tolerance asked for."""
    b = synth.gaussian_spinor(dims, 64, 2)
    lat, orc, _ = setup(dims, -1, 0.11, 1.0, 71, None)
    x, info, rc = lat.solve(to_gpu(b), tol=1e-10, **kw)
    assert rc == 0 and all(i["status"] == 0 for i in info)
    y = lat.apply(x) - to_gpu(b)
    for k in range(2):
        assert np.linalg.norm(to_host(y[k])) <= 1e-10 * np.linalg.norm(b[k])
    again, _, _ = lat.solve(to_gpu(b), tol=1e-10, **kw)
    assert np.array_equal(to_host(x), to_host(again))
    new, _, _ = setup.__wrapped__(dims, -1, 0.11, 1.0, 71, None)
    first, _, _ = new.solve(to_gpu(b), tol=1e-10, **kw)
    assert np.array_equal(to_host(x), to_host(first))


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("limit", [1, 3, 17])
def test_inner_limits_with_the_queue_length_of_the_solve_before(limit, graph):
    """An inner solve that cannot reach its tolerance runs to its limit, however
    long the first queue: 2 limit iterations for each outer one."""
    dims = (4, 4, 6, 8)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 72, None)
    b = synth.gaussian_spinor(dims, 65, 2)
    _, info, _ = lat.solve(to_gpu(b), raise_on_error=False, tol=1e-9, use_ras=0, inner_tol=1e-30, max_inner=limit,
                           max_outer=3, use_graph=graph)
    for i in info:
        assert i["outer_iters"] > 0
        assert i["inner_iters_total"] == 2 * limit * i["outer_iters"]


@pytest.mark.parametrize("outer,limit", [("FBICGSTAB", 50), ("DC", 100), ("PLAIN64_EO", 500), ("PLAIN64", 500),
                                         ("FBICGSTAB", 1), ("DC", 1), ("PLAIN64_EO", 3)])
@pytest.mark.parametrize("warm", [0, 1])
def test_reported_residual_is_that_of_the_solution(outer, limit, warm):
    """true_relres and status belong to the x returned, converged or stopped at the
    limit; the operator's rounding is a few 1e-16 of |b| in either computation."""
    from paper_1612_06556_amd import wcl
    dims = (6, 4, 8, 10)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 73, None)
    b = synth.gaussian_spinor(dims, 66, 3)
    b[1] = 0.0
    kw = dict(raise_on_error=False, tol=1e-10, outer=getattr(wcl, "OUTER_" + outer), max_outer=limit, use_ras=0, inner_tol=0.1)
    if warm:
        kw["x0"] = lat.solve(to_gpu(b), tol=1e-10)[0]
        kw["x0"][2] *= 1.001
    x, info, _ = lat.solve(to_gpu(b), **kw)
    r = to_host(lat.apply(x)) - b
    for k in (0, 2):
        rel_k = np.linalg.norm(r[k]) / np.linalg.norm(b[k])
        print(outer, limit, warm, k, info[k]["true_relres"], rel_k, info[k]["status"], flush=True)
        assert abs(info[k]["true_relres"] - rel_k) <= 1e-14 + 1e-9 * rel_k
        assert (info[k]["status"] == 0) == (rel_k <= 1e-10)
    assert not to_host(x[1]).any()
