"""Applications recorded in a caller's graph (any operator, any number of
right-hand sides): the workspace they were recorded with stays theirs, and what
is missing is allocated while recording."""
import pytest

from gpu_util import require_gpu, to_gpu
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu

# both sides of the 32768 half-sites where D in FP16 and Dhat change their route
CASES = [("D", 16, (16, 16, 16, 32)), ("HOP", 16, (16, 16, 16, 32)), ("SCHUR", 32, (8, 8, 8, 8)),
         ("SCHUR", 64, (16, 16, 16, 32)), ("SCHUR_RHS", 64, (8, 8, 8, 8)), ("RAS", 32, (8, 8, 8, 8)),
         ("SAP", 32, (8, 8, 8, 8))]


def _lattice(name, dims):
    torch = require_gpu()
    from paper_1612_06556_amd import wcl
    lat = wcl.Lattice(dims)
    lat.set_gauge(torch.from_numpy(synth.su3_field(dims, 87)).cuda())
    lat.set_params(0.12, 1.0)
    lat.set_ras(1, 4, 0, 1 if name == "SAP" else 0)
    return lat, getattr(wcl, "OP_" + ("RAS" if name == "SAP" else name))


def _record(lat, op, psi, prec):
    torch = require_gpu()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = lat.apply_op(op, psi, prec=prec)
    return graph, out


def _replays(graph, out, want):
    torch = require_gpu()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert bool((out == want).all())


@pytest.mark.parametrize("name,prec,dims", CASES)
def test_recorded_workspace_outlives_larger_calls(name, prec, dims):
    """Recorded with one right-hand side, replayed after eager calls with more,
    whose workspace is larger (and other allocations since)."""
    torch = require_gpu()
    lat, op = _lattice(name, dims)
    psi = to_gpu(synth.gaussian_spinor(dims, 88, 5))
    want = lat.apply_op(op, psi[0], prec=prec)
    graph, out = _record(lat, op, psi[0], prec)
    for n in (2, 3, 5):
        got = lat.apply_op(op, psi[:n], prec=prec)
        junk = torch.full((n << 20,), float("nan"), dtype=torch.float64, device="cuda")
        assert bool((got[0] == want).all())
        _replays(graph, out, want)
        del junk
    lat.close()


# what was applied before decides which buffers exist: none, or another tier's
BEFORE = [None, ("D", 64)]


@pytest.mark.parametrize("name,prec,dims", CASES)
@pytest.mark.parametrize("before", BEFORE)
def test_recorded_first_or_with_more_right_hand_sides(name, prec, dims, before):
    """The first application of its kind only recorded, then one with more
    right-hand sides than any before."""
    from paper_1612_06556_amd import wcl
    psi = to_gpu(synth.gaussian_spinor(dims, 89, 3))
    ref, op = _lattice(name, dims)
    want = ref.apply_op(op, psi, prec=prec)
    ref.close()
    lat, op = _lattice(name, dims)
    if before:
        lat.apply_op(getattr(wcl, "OP_" + before[0]), psi[0], prec=before[1])
    g1, out1 = _record(lat, op, psi[0], prec)
    g3, out3 = _record(lat, op, psi, prec)
    _replays(g3, out3, want)
    _replays(g1, out1, want[0])
    lat.close()
