"""The coarse GMRES with one workgroup per rhs at every width of its vectors
and the many-workgroup one beyond: a V-cycle with a fixed number of coarse
iterations over a restart, in FP32 (and FP16 storage) against FP64, whose
bound between the two paths is lower, so that neighbouring widths check each
other.  The FP64 V-cycle itself is checked against the oracle elsewhere."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# elements per coarse vector (blocks * ntv): 3072 and 6144 (4 and 8 per
# thread), 12288 (16), 20480 (24 in FP32, many workgroups in FP64), 32768
# (many workgroups in both); 17 rhs take the matrix-core stencils
@pytest.mark.parametrize("L,ntv,nrhs", [((8, 8, 8, 8), 12, 3), ((8, 8, 8, 8), 24, 5), ((8, 8, 8, 16), 24, 1),
                                        ((8, 8, 16, 16), 20, 2), ((8, 8, 16, 16), 32, 1)])
def test_vcycle_widths(L, ntv, nrhs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    U = torch.from_numpy(synth.su3_field(L, 0.4, 831)).cuda()
    tv = torch.from_numpy(synth.gaussian_spinors(L, ntv, 832)).cuda()
    y = torch.from_numpy(synth.gaussian_spinors(L, nrhs, 833)).cuda()
    y[nrhs - 1] *= 1e-3
    xs = []
    for prec in (dd.FP64, dd.FP32, dd.MIXED16):
        p = dd.default_params(L=L, block=(2, 2, 2, 2), m0=-0.1, ntv=ntv, prec=prec, max_rhs=nrhs, coarse_restart=3,
                              coarse_fixed_its=5)
        ctx = dd.Context(p, U)
        ctx.import_tv(tv)
        x = torch.empty_like(y)
        ctx.mg_apply(x, y, nrhs)
        xs.append(x)
        ctx.close()
    for x, tol in ((xs[1], 1e-5), (xs[2], 1e-2)):  # the parity bars of the V-cycle
        err = float(((x - xs[0]).abs().amax(dim=(1, 2, 3, 4, 5, 6)) / xs[0].abs().amax(dim=(1, 2, 3, 4, 5, 6))).max())
        assert err <= tol, err


def test_zero_and_converged_rhs():
    """A zero rhs stops at the start of the first cycle, beside one that iterates; solutions are exact zeros."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    L = (8, 8, 8, 8)
    p = dd.default_params(L=L, block=(2, 2, 2, 2), m0=-0.1, ntv=12, prec=dd.FP32, max_rhs=3)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.4, 834)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, 12, 835)).cuda())
    y = torch.from_numpy(synth.gaussian_spinors(L, 3, 836)).cuda()
    y[1] = 0.0
    x, z = torch.empty_like(y), torch.empty_like(y[:1])
    for _ in range(3):  # calls of different rhs counts share the activity counter
        ctx.mg_apply(x, y, 3)
        ctx.mg_apply(z, y[:1].contiguous(), 1)
        assert bool((x[1] == 0).all())
        err = float((z[0] - x[0]).abs().max() / x[0].abs().max())
        assert err <= 1e-5, err
    ctx.close()
