"""The orthonormalisation of the test vectors on the aggregates at the edges
of its tiles: one to eight steps of four vectors, full and ragged, one to
three Gram tiles, blocks whose sites are not a multiple of 16, few aggregates
(their Gram matrices in parts) and many.  The stored basis equals the
oracle's unique Q (relative to the largest element: FP64 1e-12, FP32 1e-5,
FP16 storage 1e-2), and after vectors that are linearly dependent on an
aggregate, which are refused, the context holds no setup until the next."""
import numpy as np
import pytest

import synth
from oracle import coarse, sap

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2}


def _ctx(L, block, ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    p = dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=(dd.FP64, dd.FP32, dd.MIXED16)[prec], max_rhs=1)
    return dd, dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.4, 871)).cuda())


@pytest.mark.parametrize("L,block,ntv", [((4, 4, 4, 4), (2, 2, 2, 2), 1), ((6, 4, 4, 4), (3, 2, 2, 2), 5),
                                         ((8, 8, 8, 8), (4, 4, 4, 4), 16), ((4, 6, 4, 6), (2, 3, 2, 3), 17),
                                         ((8, 4, 8, 4), (4, 2, 4, 2), 24), ((4, 4, 10, 4), (2, 2, 5, 2), 28),
                                         ((8, 8, 8, 8), (2, 2, 2, 2), 32)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_basis_matches_oracle(L, block, ntv, prec):
    dd, ctx = _ctx(L, block, ntv, prec)
    tv = synth.gaussian_spinors(L, ntv, 872)
    ctx.import_tv(torch.from_numpy(tv).cuda())
    ref = coarse.orthonormalise(sap.Blocking(L, block), tv)
    W = torch.empty((ntv,) + tuple(reversed(L)) + (4, 3), dtype=torch.complex128, device="cuda")
    ctx.export_basis(W)
    assert np.abs(W.cpu().numpy() - ref).max() <= TOL[prec] * np.abs(ref).max()
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_dependent_vectors_are_refused(prec):
    L = (4, 4, 4, 4)
    dd, ctx = _ctx(L, (2, 2, 2, 2), 6, prec)
    tv = torch.from_numpy(synth.gaussian_spinors(L, 6, 873)).cuda()
    ctx.import_tv(tv)
    first, again = torch.empty_like(tv), torch.empty_like(tv)
    ctx.export_basis(first)
    bad = tv.clone()
    bad[4] = 0.0
    with pytest.raises(dd.DDAMGError):
        ctx.import_tv(bad)
    with pytest.raises(dd.DDAMGError):
        ctx.export_basis(again)
    ctx.import_tv(tv)
    ctx.export_basis(again)
    assert torch.equal(first, again)
    ctx.close()
