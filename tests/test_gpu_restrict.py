"""Restriction at the edges of its kernels: one, two and up to four rhs
(vector units, the test vectors shared out over workgroups), five and more
(matrix cores: tiles of 16 test vectors and 16 or 32 rhs, runs of 16 sites),
against the sum over the exported basis."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def restrict(W, y, L, b):
    """sum over each block's sites and the components of each chirality of conj(W_a) y_r"""
    def agg(f):
        n = f.shape[0]
        f = f.reshape(n, L[3] // b[3], b[3], L[2] // b[2], b[2], L[1] // b[1], b[1], L[0] // b[0], b[0], 2, 6)
        f = f.transpose(1, 3, 5, 7, 9, 0, 2, 4, 6, 8, 10)
        return f.reshape(-1, 2, n, b[0] * b[1] * b[2] * b[3] * 6)
    A, Y = agg(W), agg(y)
    return np.einsum('bhak,bhrk->rbha', np.conj(A), Y)


# blocks of 90 and 24 sites (a run of 16 cut short), 16 (one run, one wave), 256
@pytest.mark.parametrize("L,block,ntv", [((6, 10, 4, 6), (3, 5, 2, 3), 17), ((6, 4, 4, 4), (3, 2, 2, 2), 6),
                                         ((4, 4, 4, 8), (2, 2, 2, 2), 16), ((8, 8, 8, 8), (4, 4, 4, 4), 24),
                                         ((4, 4, 8, 8), (2, 2, 4, 4), 32)])
@pytest.mark.parametrize("prec", (0, 1, 2))
def test_restrict_edges(L, block, ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    p = dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=prec, max_rhs=33)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.3, 841)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, ntv, 842)).cuda())
    W = torch.empty(ntv, L[3], L[2], L[1], L[0], 4, 3, dtype=torch.complex128, device="cuda")
    ctx.export_basis(W)
    y = synth.gaussian_spinors(L, 33, 843)
    y[1] *= 1e-5
    ref = restrict(W.cpu().numpy(), y, L, block)
    nb = ref.shape[1]
    for nrhs in (1, 2, 3, 4, 5, 16, 17, 33):
        out = torch.full((nrhs, nb, 2, ntv), 3.0, dtype=torch.complex128, device="cuda")
        ctx.mg_restrict(out, torch.from_numpy(np.ascontiguousarray(y[:nrhs])).cuda(), nrhs)
        o = out.cpu().numpy()
        for r in range(nrhs):
            err = np.abs(o[r] - ref[r]).max() / np.abs(ref[r]).max()
            assert err <= (1e-12 if prec == 0 else 1e-5), (nrhs, r, err)
    ctx.close()
