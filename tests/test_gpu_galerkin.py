"""The block-crossing couplings of D_c on the matrix cores at the edges of
their tiles: one to four tiles of 16 of the 2 N_tv rows, full and ragged, and
faces that do not fill a chunk of eight (four) sites, against the oracle.
Tolerances relative to the largest element: FP64 1e-12, FP32 1e-5, FP16
storage 1e-2 (the parity bars of the coarse operator)."""
import numpy as np
import pytest

import synth
from oracle import coarse, dirac, sap

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2}


@pytest.mark.parametrize("L,block,ntv", [((4, 4, 4, 4), (2, 2, 2, 2), 1), ((4, 4, 4, 4), (2, 2, 2, 2), 8),
                                         ((6, 4, 4, 4), (3, 2, 2, 2), 9), ((4, 6, 4, 6), (2, 3, 2, 3), 17),
                                         ((4, 4, 8, 4), (2, 2, 4, 2), 24), ((6, 4, 4, 4), (3, 2, 2, 2), 25),
                                         ((4, 4, 4, 4), (2, 2, 2, 2), 32)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_couplings_match_oracle(L, block, ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    U = synth.su3_field(L, 0.4, 861)
    blk = sap.Blocking(L, block)
    W = coarse.orthonormalise(blk, synth.gaussian_spinors(L, ntv, 862))
    p = dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=(dd.FP64, dd.FP32, dd.MIXED16)[prec], max_rhs=1)
    ctx = dd.Context(p, torch.from_numpy(U).cuda())
    ctx.import_basis(torch.from_numpy(np.ascontiguousarray(W)).cuda())
    ref = coarse.coarse_operator(U, dirac.clover_term(U, -0.1, 1.0), blk, W)
    D = torch.zeros((blk.nblocks, 9, 2 * ntv, 2 * ntv), dtype=torch.complex128, device="cuda")
    ctx.export_coarse(D)
    assert np.abs(D.cpu().numpy() - ref).max() <= TOL[prec] * np.abs(ref).max()
    ctx.close()
