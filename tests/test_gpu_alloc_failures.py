"""A failed allocation of a workspace: the call reports it, and the next one
allocates what is missing instead of taking the workspace as whole.  Every
allocation of a call is refused once in turn (through the allocator hook);
the call then succeeds with the result of a context that met no failure."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L, BLOCK, NTV = (8, 8, 8, 8), (4, 4, 4, 4), 4
ENOMEM = -4


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Allocator:
    """hipMalloc of torch's allocator; refuses allocation number fail_at."""

    def __init__(self):
        self.count, self.fail_at = 0, None

    def alloc(self, n):
        self.count += 1
        if self.count == self.fail_at:
            return 0
        return torch.cuda.caching_allocator_alloc(n)

    def free(self, ptr):
        torch.cuda.caching_allocator_delete(ptr)

    def arm(self, k):
        self.count, self.fail_at = 0, k


@pytest.fixture
def hooked():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    a = Allocator()
    dd.set_allocator(a.alloc, a.free)
    yield dd, a
    dd.set_allocator()


@pytest.mark.parametrize("prec", (0, 1, 2))
def test_setup_workspace(hooked, prec):
    """mg_setup: its smoother and D_c work in buffers of the first setup."""
    dd, a = hooked
    U, tv = dev(synth.su3_field(L, 0.4, 901)), dev(synth.gaussian_spinors(L, NTV, 902))
    y = dev(synth.gaussian_spinors(L, 1, 903))
    p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=NTV, prec=prec, max_rhs=1, n_setup=1)
    ref = dd.Context(p, U)
    ref.mg_setup(tv)
    want, got = torch.empty_like(y), torch.empty_like(y)
    ref.mg_apply(want, y, 1)
    ref.close()
    refused = 0
    for k in range(1, 20):
        ctx = dd.Context(p, U)
        a.arm(k)
        try:
            ctx.mg_setup(tv)
            done = True
        except dd.DDAMGError as e:
            assert e.code == ENOMEM
            done = False
            refused += 1
        a.arm(None)
        if not done:
            ctx.mg_setup(tv)
        ctx.mg_apply(got, y, 1)
        assert torch.equal(got, want), k
        ctx.close()
        if done:
            break
    assert refused >= 4


def test_outer_workspace(hooked):
    """solve: the outer basis and vectors, at the first solve and when more rhs come."""
    dd, a = hooked
    U, tv = dev(synth.su3_field(L, 0.4, 911)), dev(synth.gaussian_spinors(L, NTV, 912))
    f = dev(synth.gaussian_spinors(L, 3, 913))
    p = dd.default_params(L=L, block=BLOCK, m0=-0.1, ntv=NTV, prec=1, max_rhs=3, n_setup=1)

    def solve(ctx, n):
        u = torch.zeros_like(f[:n])
        code, _ = ctx.solve(u, f[:n].contiguous(), n, 1e-10)
        assert code == dd.OK
        return u
    ref = dd.Context(p, U)
    ref.mg_setup(tv)
    want = {n: solve(ref, n) for n in (1, 3)}
    ref.close()
    for first in (1, 3):
        refused = 0
        for k in range(1, 60):
            ctx = dd.Context(p, U)
            ctx.mg_setup(tv)
            if first == 1:
                solve(ctx, 1)
            a.arm(k)
            try:
                solve(ctx, 3)
                done = True
            except dd.DDAMGError as e:
                assert e.code == ENOMEM
                done = False
                refused += 1
            a.arm(None)
            for n in (1, 3):  # fewer rhs than the call that failed, then as many
                u = solve(ctx, n)
                assert float((u - want[n]).abs().max() / want[n].abs().max()) <= 1e-8, (k, n)
            ctx.close()
            if done:
                break
        assert refused >= 10


def test_staging(hooked):
    """dirac_apply on overlapping fields: its two staging buffers grow with nrhs."""
    dd, a = hooked
    U = dev(synth.su3_field(L, 0.4, 921))
    buf = dev(synth.gaussian_spinors(L, 3, 922))
    ctx = dd.Context(dd.default_params(L=L, block=BLOCK, ntv=NTV, prec=1, max_rhs=2), U)
    want = torch.empty_like(buf[:1])
    ctx.dirac_apply(want, buf[:1].contiguous(), 1, dd.FP64)

    def shifted(n):
        b = buf.clone()
        half = b[0].numel() // 2  # out starts in the middle of in
        flat = b.view(-1)
        inp, out = flat[:n * b[0].numel()], flat[half:half + n * b[0].numel()]
        ctx.dirac_apply(out, inp, n, dd.FP64)
        return out[:b[0].numel()].view_as(want)
    err = lambda x: float((x - want).abs().max() / want.abs().max())
    assert err(shifted(1)) <= 1e-13
    for k in (1, 2):
        a.arm(k)
        with pytest.raises(dd.DDAMGError) as e:
            shifted(2)
        assert e.value.code == ENOMEM
        a.arm(None)
        assert err(shifted(1)) <= 1e-13
    assert err(shifted(2)) <= 1e-13
    ctx.close()


def test_network_workspace(hooked):
    """ddamg_net: the activations of proposals and the gradients of training."""
    dd, a = hooked
    ctx = dd.Context(dd.default_params(L=L, block=BLOCK, ntv=NTV, prec=1, max_rhs=1), dev(synth.su3_field(L, 0.4, 931)))
    ctx.import_tv(dev(synth.gaussian_spinors(L, NTV, 932)))
    noise = dev(synth.gaussian_spinors(L, 2, 933))
    net = dd.Net((2, 3, NTV))
    w = torch.randn(net.nw, 2, generator=torch.Generator().manual_seed(9)).cuda() * 0.3
    net.set_weights(torch.view_as_complex(w).contiguous())
    out, want = (torch.empty(NTV, *noise.shape[1:], dtype=torch.complex128, device="cuda") for _ in range(2))
    a.arm(1)
    with pytest.raises(dd.DDAMGError) as e:
        net.propose(ctx, out, noise)
    assert e.value.code == ENOMEM
    a.arm(None)
    net.propose(ctx, out, noise)
    assert bool(torch.isfinite(torch.view_as_real(out)).all())
    losses = []
    for k in (None, 1, 2, 3, 4, 5):
        n2 = dd.Net((2, 3, NTV))
        n2.set_weights(torch.view_as_complex(w).contiguous())
        if k:
            a.arm(k)
            with pytest.raises(dd.DDAMGError) as e:
                n2.add_sample(ctx)
            assert e.value.code == ENOMEM
            a.arm(None)
        loss, grad = n2.loss_grad(n2.add_sample(ctx), noise)
        losses.append(loss)
        n2.propose(ctx, want, noise)
        assert torch.equal(out, want)
        n2.close()
    assert all(x == losses[0] for x in losses)
    net.close()
    ctx.close()
