"""The smoother's carried residual over many phases: V-cycles of 16 iterations
against the oracle, which forms y - D x anew in every phase, and a setup of 16
smoother passes against FP64's."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BLOCK = (4, 4, 4, 4)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def relerr(a, b):
    return float((a - b).abs().max() / b.abs().max())


def test_vcycle_of_16():
    """Each of the 128 minimal-residual updates of a block rounds its carried
    residual once, which D^-1 (condition below 100 here) turns into an error of the
    solution: 6e-8 sqrt(128) 100, that is 1e-4, in FP32; FP64 keeps the V-cycle's
    parity bar."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    from oracle import mg
    L, ntv = (8, 8, 8, 8), 4
    U = synth.su3_field(L, 0.4, 871)
    y = synth.gaussian_spinors(L, 1, 872)
    tv = synth.gaussian_spinors(L, ntv, 873)
    M = mg.MG(mg.Params(L, BLOCK, -0.1, 1.0, ntv, coarse_fixed_its=4, nu=16), U)
    for prec, tol in ((dd.FP64, 1e-12), (dd.FP32, 1e-4)):
        p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=ntv, prec=prec, max_rhs=1, nu=16, coarse_fixed_its=4)
        ctx = dd.Context(p, dev(U))
        ctx.import_tv(dev(tv))
        if M.W is None:
            W = torch.empty(ntv, L[3], L[2], L[1], L[0], 4, 3, dtype=torch.complex128, device="cuda")
            ctx.export_basis(W)
            M.set_basis(W.cpu().numpy())
            ref = M.vcycle(y[0])
        x = torch.empty_like(dev(y))
        ctx.mg_apply(x, dev(y), 1)
        assert np.abs(x.cpu().numpy()[0] - ref).max() / np.abs(ref).max() <= tol
        ctx.close()


def test_setup_of_16_passes():
    """The parity bar of one pass (1e-5 in FP32, 1e-2 with FP16 storage) for each of them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    L = (8, 8, 8, 16)
    U = dev(synth.su3_field(L, 0.4, 874))
    for ntv in (4, 20):
        tv0 = dev(synth.gaussian_spinors(L, ntv, 875))
        out = []
        for prec in (dd.FP64, dd.FP32, dd.MIXED16):
            p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=ntv, prec=prec, max_rhs=1, init_passes=16, n_setup=0)
            ctx = dd.Context(p, U)
            tv = torch.empty_like(tv0)
            ctx.mg_setup(tv0)
            ctx.export_tv(tv)
            out.append(tv)
            ctx.close()
        assert relerr(out[1], out[0]) <= 16e-5
        assert relerr(out[2], out[0]) <= 16e-2
