"""Operators on canonical spinors (one launch, both parities, every
right-hand side) and the batched layout conversions, at the sizes where a
workgroup's group of site pairs can go wrong: lattices whose half volume is
not a multiple of the group (32 or 128 pairs), tiles smaller and larger than
it, one and several right-hand sides."""
import numpy as np
import pytest

from gpu_util import rel, setup, site_err, to_gpu, to_host
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu

# the storage tiers' bounds of test_gpu_ops; per site ten times those
TOL = {64: 1e-13, 32: 1e-6, 16: 3e-3}

SHAPES = [
    ((6, 6, 6, 6), None, 1),         # 648 pairs: 20 groups of 32 and one of 8; 2^4 tiles
    ((4, 4, 4, 4), (4, 4, 4, 4), 3),  # every neighbour inside the 128 pairs
    ((10, 14, 18, 26), None, 2),     # 32760 pairs x 2: groups of 128, the last of 120
    ((8, 8, 8, 16), (8, 4, 8, 4), 9),  # x-row tiles of 512 pairs, 36864 pairs in all
]


def _reference(orc, name, v):
    if name in ("D", "DDAG"):
        return orc.D(v, name == "DDAG")
    out = {"HOP": orc.hop, "CLOVER": orc.clover, "CLOVER_INV": orc.clover_inv, "SCHUR": orc.schur,
           "SCHUR_RHS": orc.schur_rhs}[name](v)
    return out


@pytest.mark.parametrize("dims,tile,nrhs", SHAPES)
@pytest.mark.parametrize("name", ["D", "DDAG", "HOP", "CLOVER", "CLOVER_INV", "SCHUR", "SCHUR_RHS"])
def test_canonical_ops(dims, tile, nrhs, name):
    from paper_1612_06556_amd import wcl
    lat, orc, _ = setup(dims, -1, 0.12, 1.0, 77, tile)
    psi = synth.gaussian_spinor(dims, 78, nrhs)
    ref = [_reference(orc, name, psi[k]) for k in (0, nrhs - 1)]
    op = getattr(wcl, "OP_" + name)
    for comp in (0, 1):
        lat.set_compression(comp)
        for prec in ((64,) if name == "SCHUR_RHS" else (64, 32, 16)):
            out = lat.apply_op(op, to_gpu(psi), prec=prec)
            one = lat.apply_op(op, to_gpu(psi[nrhs - 1]), prec=prec)
            assert np.array_equal(to_host(out[nrhs - 1]), to_host(one))
            for k, r in zip((0, nrhs - 1), ref):
                e, es = rel(to_host(out[k]), r), site_err(to_host(out[k]), r)
                print(name, dims, prec, comp, f"{e:.2e} {es:.2e}", flush=True)
                assert e <= TOL[prec] and es <= 10 * TOL[prec]
    lat.set_compression(0)


@pytest.mark.parametrize("prec", [64, 32, 16])
def test_nonfinite_stays_local(prec):
    """A NaN at one site reaches that site and its eight neighbours only."""
    dims = (8, 8, 8, 8)
    lat, _, _ = setup(dims, -1, 0.12, 1.0, 1001, None)
    psi = synth.gaussian_spinor(dims, 5)
    n = 3 + 8 * (4 + 8 * (0 + 8 * 7))
    psi[n, 0, 0] = np.nan
    out = to_host(lat.apply(to_gpu(psi), prec=prec)).reshape(-1, 12)
    bad = set(np.nonzero(~np.isfinite(out).all(axis=1))[0])
    near = {n} | {n + d for d in (1, -1, 8, -8, 64, 7 * 64, -512, -7 * 512)}
    assert bad == near
