"""The inverse of the even self blocks of D_c at the edges of its two widths
(2 N_tv = 2, 6, 32, 34, 64) on blocks that need their rows interchanged: a
V-cycle without smoothing on an injected D_c of random unitary self blocks
with a zero diagonal start (the rows of a unitary matrix permuted; odd
blocks the identity, no couplings) solves D_c x_c = R y, so that D_c R x = R y
to FP64 rounding, 1e-12 of the largest entry.  A singular even block, also
one that only a later step meets, is refused."""
import numpy as np
import pytest

import synth
from oracle import coarse, sap

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _unitary(rng, n):
    q = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))[0]
    q[0, 0] = 0.0 if n > 2 else q[0, 0]
    return q


@pytest.mark.parametrize("ntv", [1, 3, 16, 17, 32])
def test_interchanges_and_singular_blocks(ntv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    L, block, n = (4, 4, 4, 4), (2, 2, 2, 2), 2 * ntv
    blk = sap.Blocking(L, block)
    p = dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=dd.FP64, max_rhs=2, nu=0, coarse_fixed_its=2)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.4, 881)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, ntv, 882)).cuda())
    rng = np.random.default_rng(883)
    nbr = coarse.neighbour_table(blk)
    D = np.zeros((blk.nblocks, 9, n, n), dtype=np.complex128)
    # neighbours have the other parity: two colours from block 0
    colour = -np.ones(blk.nblocks, dtype=int)
    colour[0], todo = 0, [0]
    while todo:
        b = todo.pop()
        for c in set(int(v) for v in nbr[b][1:]):
            if colour[c] < 0:
                colour[c] = 1 - colour[b]
                todo.append(c)
    for b in range(blk.nblocks):
        D[b, 0] = _unitary(rng, n) if colour[b] == 0 else np.eye(n)
    ctx.import_coarse(torch.from_numpy(D).cuda())
    y = torch.from_numpy(synth.gaussian_spinors(L, 2, 884)).cuda()
    x = torch.empty_like(y)
    ctx.mg_apply(x, y, 2)
    yc = torch.zeros((2, blk.nblocks, 2, ntv), dtype=torch.complex128, device="cuda")
    xc = torch.zeros_like(yc)
    ctx.mg_restrict(yc, y, 2)
    ctx.mg_restrict(xc, x, 2)
    yc, xc = yc.cpu().numpy().reshape(2, -1, n), xc.cpu().numpy().reshape(2, -1, n)
    got = coarse.coarse_apply(D, nbr, xc)
    assert np.abs(got - yc).max() <= 1e-12 * np.abs(yc).max()
    even = np.where(colour == 0)[0]
    for b in (even[0], even[-1]):
        bad = D.copy()
        bad[b, 0, :, n - 1] = bad[b, 0, :, 0] if n > 2 else 0.0
        if n <= 2:
            bad[b, 0] = 0.0
        else:
            bad[b, 0, :, 0] = bad[b, 0, :, n - 1] = 0.0
        with pytest.raises(dd.DDAMGError):
            ctx.import_coarse(torch.from_numpy(bad).cuda())
    ctx.close()
