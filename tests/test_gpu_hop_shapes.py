"""The hopping kernel itself, in every launch shape that the solvers, wcl_bench_hop
or the autotuner can select: its output against the FP64 oracle and, between
shapes, bitwise.  (wcl_apply and wcl_apply_op run kernels of their own on
canonical vectors, which have one shape.)"""
import ctypes
import itertools

import pytest

from gpu_util import even_mask, rel, require_gpu, setup, site_err, to_gpu, to_host
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu

# the storage tiers' bounds of the operator tests; per site ten times those
TOL = {64: 1e-13, 32: 1e-6, 16: 3e-3}
CASES = [  # dims, tbc, kappa, csw, seed, tile
    ((8, 8, 8, 8), -1, 0.12, 1.0, 1001, None),
    ((4, 6, 8, 4), -1, 0.125, 1.3, 7, None),              # 2^4 tiles, ragged last workgroup
    ((6, 4, 4, 8), 1, 0.126, 1.0, 8, (2, 2, 2, 4)),       # periodic, non-cubic tile
    ((8, 8, 8, 16), -1, 0.126, 1.0, 1005, (8, 4, 8, 4)),  # tiles spanning whole x-rows
    ((24, 24, 24, 32), -1, 0.126, 1.0, 1003, None),       # the benchmark's lattice, its two layouts
    ((24, 24, 24, 32), -1, 0.126, 1.0, 1003, (24, 4, 8, 4)),
]
# block, depth, xcd, nt, stage, site blocks per workgroup
SHAPES = [s + (1,) for s in itertools.product((64, 128, 256), (2, 3), (0, 1), (0, 1), (1, 0))]
SHAPES += [s + (t,) for s in itertools.product((64, 128, 256), (2, 3), (0, 1), (0, 1), (1,)) for t in (2, 4, 8)]

_refs = {}


def _reference(case, orc, psi, pe):
    if case[0] not in _refs:
        _refs.clear()
        _refs[case[0]] = {"H": orc.hop(psi), "Dhat": orc.schur(pe), "D": orc.D(psi)}
    return _refs[case[0]]


def _ids(c):
    return "x".join(map(str, c[0])) + ("_tile" + "x".join(map(str, c[5])) if c[5] else "")


def _hop(lat, op, psi, lp, vp, dots=0):
    from paper_1612_06556_amd import wcl
    lib = wcl.load()
    call = lib.wclt_hop
    call.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p] + [ctypes.c_int] * 4
    psi, nrhs = lat._spinors(psi)
    out = require_gpu().empty_like(psi)
    lat._sync_stream()
    wcl._check(call(lat.h, op, psi.data_ptr(), out.data_ptr(), nrhs, lp, vp, dots))
    return out


def _shape(lat, block=256, depth=2, xcd=1, nt=0, stage=1, tpw=1, rpt=1):
    from paper_1612_06556_amd import wcl
    wcl.wcl_set_tuning(lat.h, block, depth, xcd, nt)
    wcl.wcl_set_hop_staging(lat.h, stage)
    wcl.wcl_set_hop_tiles(lat.h, tpw)
    wcl.wcl_set_batch_tuning(lat.h, rpt)


def _launches():
    from paper_1612_06556_amd import wcl
    return [("H", wcl.OP_HOP, 32, 32), ("H", wcl.OP_HOP, 16, 32), ("Dhat", wcl.OP_SCHUR, 64, 64), ("Dhat", wcl.OP_SCHUR, 32, 32),
            ("Dhat", wcl.OP_SCHUR, 16, 32), ("Dhat", wcl.OP_SCHUR, 16, 16), ("D", wcl.OP_D, 64, 64)]


def _inputs(dims, seed, nrhs):
    psi = synth.gaussian_spinor(dims, seed, nrhs)
    pe = psi.copy()
    pe[:, ~even_mask(dims)] = 0
    return psi, pe


def _check(out, ref, prec, tag):
    e, es = rel(out, ref), site_err(out, ref)
    print(tag, f"{e:.2e} {es:.2e}", flush=True)
    assert e <= TOL[prec] and es <= 10 * TOL[prec], tag


@pytest.mark.parametrize("case", CASES, ids=_ids)
@pytest.mark.parametrize("comp", [0, 1])
def test_every_shape(case, comp):
    """One and three right-hand sides (two on the largest): the first shape against
    the oracle, the others bitwise the first; with the solver's inner products
    bitwise without them."""
    dims, tbc, kappa, csw, seed, tile = case
    lat, orc, _ = setup(dims, tbc, kappa, csw, seed, tile)
    nrhs = 2 if dims[0] == 24 else 3
    psi, pe = _inputs(dims, seed + 21, nrhs)
    ref = _reference(case, orc, psi[0], pe[0])
    lat.set_compression(comp)
    try:
        for name, op, lp, vp in _launches():
            g = to_gpu(pe if name == "Dhat" else psi)
            first = None
            for shape in SHAPES:
                _shape(lat, *shape)
                one, many = _hop(lat, op, g[0], lp, vp), _hop(lat, op, g, lp, vp)
                if first is None:
                    first = many
                    _check(to_host(many[0]), ref[name], lp, (name, dims, comp, lp, vp))
                assert bool((many == first).all()) and bool((one == first[0]).all()), (name, lp, vp, shape)
            if name == "Dhat":
                for block, stage, dots in itertools.product((64, 128, 256), (0, 1), (1, 2)):
                    _shape(lat, block=block, stage=stage)
                    assert bool((_hop(lat, op, g, lp, vp, dots) == first).all()), (lp, vp, block, stage, dots)
    finally:
        _shape(lat)
        lat.set_compression(0)


@pytest.mark.parametrize("case", CASES[:4], ids=_ids)
@pytest.mark.parametrize("comp", [0, 1])
def test_right_hand_sides_per_thread(case, comp):
    """2 or 4 right-hand sides a thread, with full and part-filled groups, each
    against the oracle."""
    dims, tbc, kappa, csw, seed, tile = case
    lat, orc, _ = setup(dims, tbc, kappa, csw, seed, tile)
    psi, pe = _inputs(dims, seed + 22, 5)
    ref = [(orc.hop(psi[k]), orc.schur(pe[k])) for k in range(5)]
    lat.set_compression(comp)
    try:
        for name, op, lp, vp in _launches():
            if vp != 32:
                continue
            g = to_gpu(pe if name == "Dhat" else psi)
            for block, xcd, rpt, nrhs in itertools.product((64, 256), (0, 1), (2, 4), (2, 3, 4, 5)):
                _shape(lat, block=block, xcd=xcd, rpt=rpt)
                out = to_host(_hop(lat, op, g[:nrhs], lp, vp))
                for k in range(nrhs):
                    r = ref[k][name == "Dhat"]
                    assert rel(out[k], r) <= TOL[lp] and site_err(out[k], r) <= 10 * TOL[lp], (name, lp, block, rpt, nrhs, k)
    finally:
        _shape(lat)
        lat.set_compression(0)
