"""The outer FGMRES where its Gram-Schmidt changes form: cycles that end
within the deferred passes (restart 3), at their last step (24 and 25 basis
vectors) and in the two-pass steps beyond, for right-hand sides that stop at
different steps, one of them zero, from zero and from nonzero initial
guesses.  A solution is accepted by its true residual in FP64, |f - D u| <=
1.01 tol |f| (the solver's own test up to the rounding of the norms)."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-10


@pytest.mark.parametrize("restart", [3, 23, 24, 40])
@pytest.mark.parametrize("guess", [False, True])
def test_outer_restart_lengths(restart, guess):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    L = (8, 4, 4, 8)
    # a weak preconditioner (one SAP sweep, one coarse step): some forty outer steps
    p = dd.default_params(L=L, block=(2, 2, 2, 2), m0=-0.2, ntv=4, prec=dd.FP32, max_rhs=4, n_setup=0, nu=1, n_mr=1,
                          coarse_fixed_its=1, outer_restart=restart)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.4, 851)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, 4, 852)).cuda())
    f = torch.from_numpy(synth.gaussian_spinors(L, 4, 853)).cuda()
    f[1] = 0.0
    f[2] *= 1e-6
    u = torch.from_numpy(synth.gaussian_spinors(L, 4, 854)).cuda() if guess else torch.zeros_like(f)
    if guess:
        u[2] *= 1e-6
        u[3] = 0.0
    rc, st = ctx.solve(u, f, 4, TOL)
    assert rc == 0
    du = torch.empty_like(u)
    ctx.dirac_apply(du, u, 4, dd.FP64)
    assert bool((u[1] == 0).all())
    for r in (0, 2, 3):
        assert float((f[r] - du[r]).norm()) <= 1.01 * TOL * float(f[r].norm())
    ctx.close()
