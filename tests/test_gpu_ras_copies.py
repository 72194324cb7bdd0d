"""The fused Schwarz kernel reads copies of the operator in its own order: they
follow every change of what they were made from."""
import pytest

from gpu_util import rel, require_gpu, to_gpu, to_host
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,core", [((8, 8, 8, 8), 4), ((6, 8, 10, 4), 2), ((8, 12, 8, 16), 4)])
def test_copies_follow_the_fields(dims, core):
    """RAS against the oracle (FP32 1e-5, FP16 3e-3) after each change: overlap
    parity there and back, kappa alone, the gauge field, link storage, tier."""
    import oracle
    from paper_1612_06556_amd import wcl
    torch = require_gpu()
    psi = synth.gaussian_spinor(dims, 12)
    U = [synth.su3_field(dims, s) for s in (13, 14)]
    lat = wcl.Lattice(dims)

    def check(kappa, u, overlap):
        orc = oracle.Oracle(dims, -1, kappa, 1.0, U[u])
        ref = orc.ras(psi, (core,) * 4, overlap, 4)
        lat.set_ras(overlap, 4)
        for comp in (0, 1):
            lat.set_compression(comp)
            for prec, tol in ((32, 1e-5), (16, 3e-3), (32, 1e-5)):
                e = rel(to_host(lat.apply_op(wcl.OP_RAS, to_gpu(psi), prec=prec)), ref)
                print(dims, kappa, u, overlap, comp, prec, f"{e:.2e}", flush=True)
                assert e <= tol

    lat.set_gauge(torch.from_numpy(U[0]).cuda())
    lat.set_params(0.12, 1.0)
    for overlap in (1, 0, 1):
        check(0.12, 0, overlap)
    lat.set_params(0.10, 1.0)
    check(0.10, 0, 1)
    lat.set_compression(0)
    lat.set_gauge(torch.from_numpy(U[1]).cuda())
    lat.set_params(0.10, 1.0)
    check(0.10, 1, 1)
    lat.close()


def test_copies_under_graph_replay():
    """A graph-replayed Schwarz solve right after a new gauge field is bitwise
    the eager one (the copies are made before the capture)."""
    from paper_1612_06556_amd import wcl
    torch = require_gpu()
    dims = (8, 8, 8, 8)
    b = to_gpu(synth.gaussian_spinor(dims, 15))
    for seed in (16, 17):
        U = torch.from_numpy(synth.su3_field(dims, seed)).cuda()
        out = []
        for graph in (1, 0):
            lat = wcl.Lattice(dims)
            lat.set_gauge(U)
            lat.set_params(0.12, 1.0)
            for _ in range(2):
                x, _, rc = lat.solve(b, use_graph=graph, inner_tol=0.1)
                assert rc == 0
                out.append(to_host(x))
            lat.close()
        assert all((x == out[0]).all() for x in out)
