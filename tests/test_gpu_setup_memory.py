"""Device memory of a setup: the FP64 field of N_tv vectors, the block operator's
columns, the D_c accumulator, with FP16 storage the dequantised basis, and no more
than 16 KiB per aggregate for the Gram-Schmidt's triangular factors."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,block,ntv", [
    ((8, 8, 8, 8), (2, 2, 2, 2), 8),
    ((8, 8, 8, 8), (2, 2, 2, 2), 32),
    ((8, 8, 8, 8), (4, 4, 4, 4), 32),   # four parts of an aggregate's Gram matrix
    ((8, 8, 8, 16), (4, 4, 4, 4), 3),
    ((6, 4, 6, 4), (3, 2, 3, 2), 17),   # two parts
])
@pytest.mark.parametrize("prec", (0, 1, 2))
def test_setup_allocates(L, block, ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    held, size = [0], {}

    def alloc(n):
        p = torch.cuda.caching_allocator_alloc(n)
        size[p] = n
        held[0] += n
        return p

    def free(p):
        held[0] -= size.pop(p)
        torch.cuda.caching_allocator_delete(p)

    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dd.set_allocator(alloc, free)
    try:
        p = dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=prec, max_rhs=1)
        ctx = dd.Context(p, dev(synth.su3_field(L, 0.4, 881)))
        before = held[0]
        ctx.mg_setup(dev(synth.gaussian_spinors(L, ntv, 882)))
        took = held[0] - before
        ctx.close()
    finally:
        dd.set_allocator()
    assert held[0] == 0
    V = L[0] * L[1] * L[2] * L[3]
    nblocks, w = V // (block[0] * block[1] * block[2] * block[3]), 16 if prec == 0 else 8
    field = ntv * 12 * V
    most = field * (16 + w + (8 if prec == 2 else 0)) + nblocks * 9 * (2 * ntv) ** 2 * w + 2 * nblocks * 16384
    assert took <= most
