"""The prolongation on both sides of each width of a pass (1, 4, 8 and 12 rhs,
full and ragged, one pass and several), test vectors that leave a remainder
in the unrolled loop, blocks that do not fill their waves, against the oracle
(relative to the largest element: FP64 1e-12, FP32 1e-5, FP16 storage 1e-2,
the parity bars of the transfer operators)."""
import numpy as np
import pytest

import synth
from oracle import coarse, sap

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2}


@pytest.mark.parametrize("L,block,ntv", [((4, 4, 4, 4), (2, 2, 2, 2), 1), ((6, 4, 4, 6), (3, 2, 2, 3), 7),
                                         ((8, 8, 8, 8), (4, 4, 4, 4), 18)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_prolong_rhs_counts(L, block, ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    blk = sap.Blocking(L, block)
    W = coarse.orthonormalise(blk, synth.gaussian_spinors(L, ntv, 892))
    p = dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=(dd.FP64, dd.FP32, dd.MIXED16)[prec], max_rhs=26)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.4, 891)).cuda())
    ctx.import_basis(torch.from_numpy(np.ascontiguousarray(W)).cuda())
    xc = synth.gaussian_coarse(blk.nblocks, ntv, 26, 893)
    ref = coarse.prolong(blk, W, xc)
    for n in (1, 2, 4, 5, 8, 9, 12, 13, 26):
        x = torch.zeros((n,) + tuple(reversed(L)) + (4, 3), dtype=torch.complex128, device="cuda")
        ctx.mg_prolong(x, torch.from_numpy(np.ascontiguousarray(xc[:n])).cuda(), n)
        assert np.abs(x.cpu().numpy() - ref[:n]).max() <= TOL[prec] * np.abs(ref[:n]).max()
    ctx.close()
