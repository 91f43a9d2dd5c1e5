"""The coarse solve of one rhs in one workgroup where its split of the
columns changes: more column groups than a slot has columns (N_tv 1), groups
that end inside a slot (N_tv 7, 10, 17, 24), 16, 32 and 64 sites, each
precision.  The V-cycle with a fixed number of coarse iterations
over restarts equals the one of the many-launch coarse solve to rounding
(FP64 1e-12, FP32 1e-5, FP16 storage 1e-4 relative to the largest element,
the bars of the two paths)."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec,L,ntv", [(0, (8, 8, 8, 8), 1), (0, (16, 8, 8, 8), 7), (1, (8, 16, 8, 8), 10),
                                        (1, (16, 8, 8, 16), 8), (1, (8, 8, 8, 8), 17), (2, (8, 8, 8, 8), 24)])
def test_single_workgroup_splits(prec, L, ntv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    names = {0: dd.FP64, 1: dd.FP32, 2: dd.MIXED16}
    p = dd.default_params(L=L, block=(4, 4, 4, 4), m0=-0.1, ntv=ntv, prec=names[prec], max_rhs=3, coarse_restart=3,
                          coarse_fixed_its=7)
    ctx = dd.Context(p, torch.from_numpy(synth.su3_field(L, 0.4, 841)).cuda())
    ctx.import_tv(torch.from_numpy(synth.gaussian_spinors(L, ntv, 842)).cuda())
    y = torch.from_numpy(synth.gaussian_spinors(L, 3, 843)).cuda()
    y[1] *= 1e-3
    y[2] = 0.0
    xs = []
    for on in (True, False):
        ctx.set_coarse_single_kernel(on)
        x = torch.empty_like(y)
        ctx.mg_apply(x, y, 3)
        xs.append(x)
    ctx.set_coarse_single_kernel(True)
    ctx.set_kernel_timing(True)
    ctx.mg_apply(torch.empty_like(y), y, 3)
    assert ctx.kernel_times()["coarse_gs"][1] == 0  # the single kernel ran
    ctx.close()
    assert bool((xs[0][2] == 0).all())
    tol = {0: 1e-12, 1: 1e-5, 2: 1e-4}[prec]
    for r in (0, 1):
        assert float((xs[0][r] - xs[1][r]).abs().max()) <= tol * float(xs[1][r].abs().max())
