"""Restriction with up to five test vectors, whose rhs beyond one pass of the
vector kernel take a second one (up to eight in FP32, four in FP64; matrix
cores above, on 2^4 blocks and for the fifth test vector), against the sum over
the exported basis."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def aggregates(f, L, b):
    n = f.shape[0]
    f = f.reshape(n, L[3] // b[3], b[3], L[2] // b[2], b[2], L[1] // b[1], b[1], L[0] // b[0], b[0], 2, 6)
    f = f.permute(1, 3, 5, 7, 9, 0, 2, 4, 6, 8, 10)
    return f.reshape(-1, 2, n, b[0] * b[1] * b[2] * b[3] * 6)


@pytest.mark.parametrize("L,block", [((6, 10, 4, 6), (3, 5, 2, 3)), ((4, 4, 4, 8), (2, 2, 2, 2)),
                                     ((8, 8, 8, 8), (4, 4, 4, 4))])
@pytest.mark.parametrize("ntv", (1, 3, 4, 5))
@pytest.mark.parametrize("prec", (0, 1, 2))
def test_restrict_few_test_vectors(L, block, ntv, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    ctx = dd.Context(dd.default_params(L=L, block=block, m0=-0.1, ntv=ntv, prec=prec, max_rhs=9),
                     torch.from_numpy(synth.su3_field(L, 0.3, 981)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, ntv, 982)).cuda())
    W = torch.empty(ntv, L[3], L[2], L[1], L[0], 4, 3, dtype=torch.complex128, device="cuda")
    ctx.export_basis(W)
    y = torch.from_numpy(synth.gaussian_spinors(L, 9, 983)).cuda()
    y[4] *= 1e-5
    Y, A = aggregates(y, L, block), aggregates(W, L, block)
    ref = torch.stack([(A.conj() * Y[:, :, r:r + 1]).sum(-1) for r in range(9)])
    for n in (2, 3, 4, 5, 8, 9):
        out = torch.full_like(ref[:n], 3.0)
        ctx.mg_restrict(out, y[:n].contiguous(), n)
        err = (out - ref[:n]).abs().amax(dim=(1, 2, 3)) / ref[:n].abs().amax(dim=(1, 2, 3))
        assert float(err.max()) <= (1e-12 if prec == 0 else 1e-5), (n, err.tolist())
    ctx.close()
