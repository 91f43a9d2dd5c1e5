"""The network with few channels, whose layers and weight gradients run on the
vector units: on a lattice that is no multiple of the 256 sites of a workgroup and
large enough for all of them, and on a smaller one where the layers of one and
two input channels do.  Proposal, loss and the gradient of every weight against
the oracle; FP32 arithmetic, 1e-5 relative to the largest element (the FP32 parity
bar of the network)."""
import numpy as np
import pytest

import synth
from oracle import sap, coarse, learned

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-5


@pytest.mark.parametrize("L,block,ch", [
    ((18, 14, 18, 16), (3, 7, 3, 4), (1, 5, 2, 4)),
    ((18, 14, 18, 16), (3, 7, 3, 4), (4, 2, 17)),
    ((12, 8, 6, 18), (3, 4, 3, 3), (2, 9, 1, 3)),
])
def test_thin_net_matches_oracle(L, block, ch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    U = synth.su3_field(L, 0.5, 621)
    blk = sap.Blocking(L, block)
    T = coarse.orthonormalise(blk, synth.gaussian_spinors(L, ch[-1], 622))
    p = dd.default_params(L=L, block=block, m0=-0.2, csw=1.0, ntv=ch[-1], prec=dd.FP64, max_rhs=2)
    ctx = dd.Context(p, torch.from_numpy(U).cuda())
    ctx.import_basis(torch.from_numpy(np.ascontiguousarray(T)).cuda())
    ws = [w.astype(np.complex64).astype(np.complex128) for w in synth.network_weights(ch, 623)]
    net = dd.Net(ch)
    net.set_weights(torch.from_numpy(np.concatenate([w.reshape(-1) for w in ws]).astype(np.complex64)).cuda())
    k = net.add_sample(ctx)
    noise = synth.gaussian_spinors(L, ch[0], 624)
    d = torch.from_numpy(np.ascontiguousarray(noise)).cuda()
    out = torch.zeros((ch[-1],) + tuple(reversed(L)) + (4, 3), dtype=torch.complex128, device="cuda")
    net.propose(ctx, out, noise=d)
    loss, g = net.loss_grad(k, noise=d)
    torch.cuda.synchronize()
    ref, _ = learned.forward(U, ws, noise)
    assert np.abs(out.cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()
    lref, gref = learned.loss_and_grad(U, ws, noise, blk, T)
    assert abs(loss - lref) <= TOL * abs(lref)
    g, o = g.cpu().numpy(), 0
    for r in gref:
        assert np.abs(g[o:o + r.size].reshape(r.shape) - r).max() <= TOL * np.abs(r).max()
        o += r.size
    net.close()
    ctx.close()
