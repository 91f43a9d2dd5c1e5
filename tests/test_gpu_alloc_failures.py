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
