"""Gauge ingest and clover build at the sizes where their regions are ragged:
extents that 4 and 8 do not divide, half volumes that 32 does not divide, and
tiles larger and smaller than a region."""
import numpy as np
import pytest

from gpu_util import rel, require_gpu, site_err, to_gpu, to_host
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,tile", [
    ((4, 4, 4, 4), None), ((6, 6, 6, 6), None), ((4, 6, 10, 14), None), ((12, 4, 20, 6), (6, 2, 10, 6)),
    ((8, 8, 8, 12), (8, 4, 8, 4)),
])
@pytest.mark.parametrize("two_row", [0, 1])
def test_clover_and_links(dims, tile, two_row):
    """T, T^-1, H after a second gauge field replaced the first: FP64 1e-13,
    FP32 1e-6, FP16 3e-3 against the oracle, per site ten times that."""
    import oracle
    from paper_1612_06556_amd import wcl
    torch = require_gpu()
    lat = wcl.Lattice(dims, -1, tile)
    lat.set_compression(two_row)
    lat.set_gauge(torch.from_numpy(synth.su3_field(dims, 5)).cuda())
    lat.set_params(0.11, 1.0)
    U = synth.su3_field(dims, 6)
    lat.set_gauge(torch.from_numpy(U).cuda())
    lat.set_params(0.12, 1.2)
    orc = oracle.Oracle(dims, -1, 0.12, 1.2, U)
    psi = synth.gaussian_spinor(dims, 7)
    for op, ref in ((wcl.OP_CLOVER, orc.clover(psi)), (wcl.OP_CLOVER_INV, orc.clover_inv(psi)), (wcl.OP_HOP, orc.hop(psi))):
        for prec, tol in ((64, 1e-13), (32, 1e-6), (16, 3e-3)):
            out = to_host(lat.apply_op(op, to_gpu(psi), prec=prec))
            assert rel(out, ref) <= tol and site_err(out, ref) <= 10 * tol
    lat.close()


@pytest.mark.parametrize("site", [0, 647, 1295])
def test_su3_check_finds_any_link(site):
    """One bad link anywhere (also in the last, ragged group) and a NaN are
    refused; the next good field is accepted."""
    from paper_1612_06556_amd import wcl
    torch = require_gpu()
    dims = (6, 6, 6, 6)
    good = synth.su3_field(dims, 8)
    lat = wcl.Lattice(dims)
    lat.set_compression(1)
    for value in (good[site, 3, 2, 1] + 1e-3, np.nan):
        bad = good.copy()
        bad[site, 3, 2, 1] = value
        with pytest.raises(wcl.WclError) as e:
            lat.set_gauge(torch.from_numpy(bad).cuda())
        assert e.value.code == wcl.WCL_EINVAL and "SU(3)" in str(e.value)
        with pytest.raises(wcl.WclError):
            lat.set_params(0.12, 1.0)
        lat.set_gauge(torch.from_numpy(good).cuda())
        lat.set_params(0.12, 1.0)
    lat.close()
