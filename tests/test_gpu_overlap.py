"""Applications whose output buffer overlaps the input: each right-hand side is
read before its result is written, one after another."""
import pytest

from gpu_util import require_gpu
from paper_1612_06556_amd import synth

pytestmark = pytest.mark.gpu

OPS = ["HOP", "CLOVER", "CLOVER_INV", "SCHUR", "SCHUR_RHS", "RAS", "D", "DDAG", "D_NOALLOC", "DDAG_NOALLOC"]


# one and several workgroups of 128 pairs, part-filled ones, FP16 on both sides of its packing limit
@pytest.mark.parametrize("dims,comp", [((4, 4, 4, 4), 0), ((6, 6, 10, 14), 1), ((16, 16, 16, 32), 0)])
@pytest.mark.parametrize("name", OPS)
def test_overlapping_buffers(dims, comp, name):
    """In place, one right-hand side further down (what was read before is
    overwritten), and half a right-hand side either way: bitwise the result in a
    buffer of its own."""
    torch = require_gpu()
    from paper_1612_06556_amd import wcl
    lat = wcl.Lattice(dims)
    lat.set_compression(comp)
    lat.set_gauge(torch.from_numpy(synth.su3_field(dims, 91)).cuda())
    lat.set_params(0.12, 1.0)
    if dims == (4, 4, 4, 4):
        lat.set_ras(0, 4)
    lat._sync_stream()
    field = lat.V * 12
    gen = torch.Generator(device="cuda")
    gen.manual_seed(92)
    buf = torch.randn(5 * field, dtype=torch.complex128, device="cuda", generator=gen)

    def call(b, src, dst, n, prec):
        i, o = b[src:].data_ptr(), b[dst:].data_ptr()
        if name.endswith("_NOALLOC"):
            wcl.wcl_apply_noalloc(lat.h, i, o, n, int(name[:4] == "DDAG"), prec)
        else:
            wcl.wcl_apply_op(lat.h, getattr(wcl, "OP_" + name), i, o, n, prec)

    precs = {"SCHUR_RHS": (64,), "RAS": (32, 16)}.get(name, (64, 32, 16))
    for prec in precs:
        for n, src, dst in ((1, field, field), (3, field, field), (3, field, 0),
                            (1, field, field + field // 2), (1, field, field - field // 2)):
            apart = torch.cat([buf, torch.zeros(n * field, dtype=buf.dtype, device="cuda")])
            call(apart, src, 5 * field, n, prec)
            b = buf.clone()
            call(b, src, dst, n, prec)
            want = buf.clone()
            want[dst:dst + n * field] = apart[5 * field:]
            assert bool((b == want).all()), (prec, n, src, dst)
    lat.close()
