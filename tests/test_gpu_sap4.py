"""The smoother on 4^4 blocks, whose residual is carried from phase to phase:
both kernels (two lanes per site on small grids, one above) against the
oracle's V-cycle, from a nonzero start (the coarse-grid correction) and, in
the setup, from zero; cycle counts with and without a carried phase; more rhs
than test vectors (the smoother's own buffers); antiperiodic faces on every
block of a lattice two blocks long."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2}  # the parity bars of the V-cycle
BLOCK = (4, 4, 4, 4)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def relerr(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("nu,n_mr", [(1, 4), (2, 3), (3, 4), (2, 0)])
@pytest.mark.parametrize("prec", (0, 1, 2))
def test_vcycle_both_kernels(nu, n_mr, prec):
    """8x8x8x16: 16 blocks per colour; up to 16 rhs run two lanes per site in
    FP32, 17 one (FP64: always one); 17 rhs exceed N_tv = 6."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    L, ntv, n = (8, 8, 8, 16), 6, 17
    U = dev(synth.su3_field(L, 0.4, 851))
    tv = dev(synth.gaussian_spinors(L, ntv, 852))
    y = dev(synth.gaussian_spinors(L, n, 853))

    def vcycle(pr, k):
        p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=ntv, prec=pr, max_rhs=k, nu=nu, n_mr=n_mr,
                              coarse_fixed_its=4)
        ctx = dd.Context(p, U)
        ctx.import_tv(tv)
        x = torch.empty_like(y[:k])
        for _ in range(2):  # the second call finds the first one's residuals and faces in the workspace
            ctx.mg_apply(x, y[:k].contiguous(), k)
        ctx.close()
        return x
    many, few = vcycle(prec, n), vcycle(prec, 3)
    ref = vcycle(dd.FP64, 2)
    assert relerr(many[:3], few) <= 2 * TOL[prec]
    assert relerr(many[:2], ref) <= TOL[prec]


def test_vcycle_oracle():
    """The carried residual against the oracle, which forms y - D x in every phase."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    from oracle import mg
    L, ntv = (8, 8, 8, 8), 4
    U = synth.su3_field(L, 0.4, 854)
    y = synth.gaussian_spinors(L, 1, 856)
    M = mg.MG(mg.Params(L, BLOCK, -0.1, 1.0, ntv, coarse_fixed_its=4), U)
    tv = synth.gaussian_spinors(L, ntv, 855)
    for prec in (dd.FP64, dd.FP32):
        p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=ntv, prec=prec, max_rhs=1, nu=3, coarse_fixed_its=4)
        ctx = dd.Context(p, dev(U))
        ctx.import_tv(dev(tv))
        if M.W is None:
            W = torch.empty(ntv, L[3], L[2], L[1], L[0], 4, 3, dtype=torch.complex128, device="cuda")
            ctx.export_basis(W)
            M.set_basis(W.cpu().numpy())
            ref = M.vcycle(y[0])
        x = torch.empty_like(dev(y))
        ctx.mg_apply(x, dev(y), 1)
        assert np.abs(x.cpu().numpy()[0] - ref).max() / np.abs(ref).max() <= TOL[prec]
        ctx.close()


@pytest.mark.parametrize("passes", (1, 2, 3))
def test_setup_from_zero(passes):
    """Initial smoother passes alone (n_setup = 0), whose sweeps start from
    zero: the test vectors of FP32 (two lanes per site for 4 vectors, one for
    20) and FP16 storage against FP64's."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    L = (8, 8, 8, 16)
    U = dev(synth.su3_field(L, 0.4, 857))
    for ntv in (4, 20):
        tv0 = dev(synth.gaussian_spinors(L, ntv, 858))
        out = []
        for prec in (dd.FP64, dd.FP32, dd.MIXED16):
            p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=ntv, prec=prec, max_rhs=1, init_passes=passes, n_setup=0)
            ctx = dd.Context(p, U)
            tv = torch.empty_like(tv0)
            for _ in range(2):
                ctx.mg_setup(tv0)
                ctx.export_tv(tv)
            out.append(tv)
            ctx.close()
        assert relerr(out[1], out[0]) <= TOL[1]
        assert relerr(out[2], out[0]) <= TOL[2]
