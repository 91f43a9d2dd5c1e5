"""dirac_apply on canonical fields, read and written in place: the two
kernels behind it (four waves per 64 sites on small lattices, staged blocks
above) against the oracle at ragged workgroups, and fields that overlap."""
import numpy as np
import pytest

import synth
from oracle import dirac

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {0: 1e-12, 1: 1e-5, 2: 1e-2}  # FP64, FP32, FP16 storage: the parity bars of the operator


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    return dd


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# (lattice, block, rhs): 768 and 4608 sites times rhs take the split kernel in
# every precision (3 * 256 + 48 sites: a ragged last workgroup), 36864 only in
# FP32, 50688 the staged one with units of 72 lanes, three per workgroup and
# two in the last
CASES = [((4, 4, 4, 4), (2, 2, 2, 2), 3), ((6, 4, 6, 6), (3, 2, 3, 1), 1), ((6, 12, 8, 8), (3, 3, 2, 4), 1),
         ((6, 12, 8, 8), (3, 3, 2, 4), 8), ((6, 12, 8, 8), (3, 3, 2, 4), 11), ((8, 8, 8, 16), (4, 4, 4, 4), 7)]


@pytest.mark.parametrize("L,block,nrhs", CASES)
def test_apply_matches_oracle(L, block, nrhs):
    dd = _gpu()
    U = synth.su3_field(L, 0.5, 811)
    A = dirac.clover_term(U, -0.2, 1.0)
    psi = synth.gaussian_spinors(L, nrhs, 812)
    ref = np.stack([dirac.apply_D(U, A, psi[r]) for r in range(nrhs)])
    ctx = dd.Context(dd.default_params(L=L, block=block, m0=-0.2, csw=1.0, ntv=1, max_rhs=nrhs), dev(U))
    x = dev(psi)
    for prec in (dd.FP64, dd.FP32, dd.MIXED16):
        out = torch.full_like(x, 5.0)
        ctx.dirac_apply(out, x, nrhs, prec)
        err = np.abs(out.cpu().numpy() - ref).max() / np.abs(ref).max()
        assert err <= TOL[prec], (prec, err)
    ctx.close()


@pytest.mark.parametrize("noalloc", (False, True))
def test_overlapping_fields(noalloc):
    """out one rhs further than in, inside one buffer: every output is that of separate buffers."""
    dd = _gpu()
    L, n = (8, 8, 8, 8), 3
    U = synth.su3_field(L, 0.5, 813)
    ctx = dd.Context(dd.default_params(L=L, block=(4, 4, 4, 4), m0=-0.2, ntv=1, max_rhs=n), dev(U))
    x = dev(synth.gaussian_spinors(L, n, 814))
    apply = ctx.dirac_apply_noalloc if noalloc else ctx.dirac_apply
    for prec in (dd.FP64, dd.MIXED16):
        ref = torch.empty_like(x)
        apply(ref, x, n, prec)
        buf = torch.zeros((n + 1,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda")
        buf[:n] = x
        apply(buf[1:], buf[:n], n, prec)
        err = float((buf[1:] - ref).abs().max() / ref.abs().max())
        assert err <= 2 * (1e-12 if prec == dd.FP64 else 1e-5), (prec, err)
    ctx.close()
