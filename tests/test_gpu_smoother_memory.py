"""Memory of the smoother on 4^4 blocks for more rhs than test vectors: none at
creation, two fields per rhs at the first call that needs them, none where
there is none to be had or while a graph is captured (the rhs then go in groups
of N_tv), and given back when a solve cannot allocate its basis."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L, NTV, NRHS = (8, 8, 8, 8), 4, 11
V = L[0] * L[1] * L[2] * L[3]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Allocator:
    """Counts what contexts hold; refuses allocation number fail_at and, if refuse is set, sizes it names."""

    def __init__(self):
        self.count, self.fail_at, self.refuse, self.held, self.size = 0, None, None, 0, {}

    def alloc(self, n):
        self.count += 1
        if self.count == self.fail_at or (self.refuse and self.refuse(n)):
            return 0
        p = torch.cuda.caching_allocator_alloc(n)
        self.size[p] = n
        self.held += n
        return p

    def free(self, ptr):
        self.held -= self.size.pop(ptr)
        torch.cuda.caching_allocator_delete(ptr)


@pytest.fixture
def hooked():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    a = Allocator()
    dd.set_allocator(a.alloc, a.free)
    yield dd, a
    dd.set_allocator()


def context(dd, prec, **more):
    p = dd.default_params(**{**dict(L=L, block=(4, 4, 4, 4), m0=-0.1, ntv=NTV, prec=prec, max_rhs=NRHS, nu=2), **more})
    return dd.Context(p, dev(synth.su3_field(L, 0.4, 991)))


def apply(ctx, y):
    x = torch.empty_like(y)
    ctx.mg_apply(x, y, y.shape[0])
    torch.cuda.synchronize()
    return x


def relerr(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("prec", (0, 1, 2))
def test_created_without(hooked, prec):
    """A context that never smooths holds no more on 4^4 blocks, whose smoother
    carries its residual, than on 4x4x4x2 ones, whose does not (and which have
    twice the coarse sites)."""
    dd, a = hooked
    held = []
    for block in ((4, 4, 4, 4), (4, 4, 4, 2)):
        ctx = context(dd, prec, block=block, ntv=1, max_rhs=32)
        held.append(a.held)
        ctx.close()
    assert held[0] <= held[1]
    assert a.held == 0


@pytest.mark.parametrize("prec", (0, 1, 2))
def test_first_call_and_none_left(hooked, prec):
    dd, a = hooked
    field = 12 * V * (16 if prec == 0 else 8)
    tv, y = dev(synth.gaussian_spinors(L, NTV, 992)), dev(synth.gaussian_spinors(L, NRHS, 993))
    ctx = context(dd, prec)
    ctx.import_tv(tv)
    few = apply(ctx, y[:NTV].contiguous())
    before = a.held
    many = apply(ctx, y)
    assert a.held == before + 2 * NRHS * field
    again = apply(ctx, y[:NTV + 1].contiguous())
    assert a.held == before + 2 * NRHS * field
    ctx.close()
    assert relerr(many[:NTV], few) <= 1e-5 and relerr(again, many[:NTV + 1]) <= 1e-5
    for k in (1, 2):  # either of the two buffers refused
        ctx = context(dd, prec)
        ctx.import_tv(tv)
        apply(ctx, y[:1].contiguous())
        before = a.held
        a.count, a.fail_at = 0, k
        got = apply(ctx, y)
        a.fail_at = None
        assert a.held == before
        assert relerr(got, many) <= (1e-13 if prec == 0 else 1e-5)
        assert relerr(apply(ctx, y), many) <= (1e-13 if prec == 0 else 1e-5)
        ctx.close()
    assert a.held == 0


def test_given_back_to_a_solve(hooked):
    """Every allocation of a solve refused once while the smoother holds its
    buffers: the solve takes them back and succeeds."""
    dd, a = hooked
    tv, f = dev(synth.gaussian_spinors(L, NTV, 992)), dev(synth.gaussian_spinors(L, NRHS, 994))
    field = 12 * V * 8

    def solve(ctx):
        u = torch.zeros_like(f)
        code, st = ctx.solve(u, f, NRHS, 1e-10)
        assert code == dd.OK and max(st["relres"]) <= 1e-10
    refused = 0
    for k in range(1, 60):
        ctx = context(dd, 1)
        ctx.mg_setup(tv)
        before = a.held
        apply(ctx, f)
        assert a.held == before + 2 * NRHS * field
        a.count, a.fail_at = 0, k
        solve(ctx)
        reached = a.count >= k
        a.fail_at = None
        refused += reached
        ctx.close()
        if not reached:
            break
    assert refused >= 10
    assert a.held == 0


def test_first_call_captured():
    """mg_apply captured by the caller before any call of so many rhs (a coarse
    lattice solved in one launch): no allocation in the capture, and replays
    with other work between them give the eager result."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    tv, y = dev(synth.gaussian_spinors(L, NTV, 992)), dev(synth.gaussian_spinors(L, NRHS, 993))
    s = torch.cuda.Stream()
    U = dev(synth.su3_field(L, 0.4, 991))
    torch.cuda.synchronize()
    ctx = dd.Context(dd.default_params(L=L, block=(4, 4, 4, 4), m0=-0.1, ntv=NTV, prec=1, max_rhs=NRHS, nu=2), U,
                     stream=s)
    ctx.import_tv(tv)
    x = torch.empty_like(y)
    ctx.mg_apply(x[:1], y[:1], 1)  # code objects loaded
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.mg_apply(x, y, NRHS)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 2 * NRHS * 12 * V * 8
    eager = torch.empty_like(y)
    for k in range(3):
        x.zero_()
        y.mul_(2.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ctx.mg_apply(eager, y, NRHS)
        torch.cuda.synchronize()
        assert relerr(x, eager) <= 1e-5, k
    ctx.close()
