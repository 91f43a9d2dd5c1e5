"""The D_c stencil at the edges of its kernels: one to four rhs (vector
units, four or two rows per lane), five and more (matrix cores, tiles of 16
rows and groups of 16 rhs), against the dense nine-slot sum with the operator
as stored."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L, BLOCK = (4, 4, 4, 6), (2, 2, 2, 1)
NB = tuple(L[i] // BLOCK[i] for i in range(4))
NBLK = NB[0] * NB[1] * NB[2] * NB[3]


def reference(D, x):
    """sum over the slots, blocks lexicographic, D [block][slot][row][col]"""
    lex = np.arange(NBLK)
    c = [lex % NB[0], lex // NB[0] % NB[1], lex // (NB[0] * NB[1]) % NB[2], lex // (NB[0] * NB[1] * NB[2])]
    out = np.einsum('bij,rbj->rbi', D[:, 0], x)
    for mu in range(4):
        for d in range(2):
            e = [v.copy() for v in c]
            e[mu] = (e[mu] + (1 if d == 0 else -1)) % NB[mu]
            nb = e[0] + NB[0] * (e[1] + NB[1] * (e[2] + NB[2] * e[3]))
            out += np.einsum('bij,rbj->rbi', D[:, 1 + 2 * mu + d], x[:, nb])
    return out


# ntv: 2 ntv rows of 2, 6 (one tile, two rows per lane), 16 and 18 (one full
# tile, a second of 2 rows), 40 and 48 (three tiles, 40 ragged), 64
@pytest.mark.parametrize("ntv", (1, 3, 8, 9, 20, 24, 32))
@pytest.mark.parametrize("prec", (0, 1, 2))
def test_stencil_edges(ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    nc = 2 * ntv
    p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=ntv, prec=prec, max_rhs=18)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.3, 821)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, ntv, 822)).cuda())
    rng = np.random.default_rng(823 + ntv)
    D = (rng.standard_normal((NBLK, 9, nc, nc)) + 1j * rng.standard_normal((NBLK, 9, nc, nc))) / np.sqrt(nc)
    D[:, 0] += 8.0 * np.eye(nc)
    ctx.import_coarse(torch.from_numpy(D).cuda())
    Ds = torch.empty(NBLK, 9, nc, nc, dtype=torch.complex128, device="cuda")
    ctx.export_coarse(Ds)
    Ds = Ds.cpu().numpy()
    # components over eight orders of magnitude, one rhs all zero
    x = synth.gaussian_coarse(NBLK, ntv, 18, 824).reshape(18, NBLK, nc)
    x *= 10.0 ** rng.uniform(-4, 4, (18, NBLK, 1))
    x[2] = 0.0
    ref = reference(Ds, x)
    for nrhs in (1, 2, 4, 5, 16, 17):
        xi = torch.from_numpy(np.ascontiguousarray(x[:nrhs])).cuda()
        out = torch.full_like(xi, 7.0)
        ctx.coarse_apply(out, xi, nrhs)
        o = out.cpu().numpy()
        for r in range(nrhs):
            s = max(np.abs(ref[r]).max(), 1e-300)
            err = np.abs(o[r] - ref[r]).max() / s
            # FP32: 9 nc products and sums of relative error 2^-22 each, at most
            assert err <= (1e-13 if prec == 0 else 9 * nc * 2.0 ** -22), (nrhs, r, err)
    ctx.close()
