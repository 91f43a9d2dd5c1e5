"""The launches of the fused coarse GMRES one by one (the library's internal
launchers, called by their C++ names): the start of a cycle, an Arnoldi step,
the end of a cycle, each against the same step in 64 bits.  A whole solve hides
a slip in one of them as further iterations."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

vp, i32, sz, f64 = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t, ctypes.c_double


class State(ctypes.Structure):  # ArnoldiState
    _fields_ = [(k, vp) for k in ("H", "cs", "sn", "g", "y", "est", "inv_h", "abstol", "active", "any", "kdone")]
    _fields_ += [("m", i32)]


class Krylov:
    """The state of `rhs` rhs at restart length m, its arrays as tensors."""

    def __init__(self, m, rhs):
        c = lambda *n: torch.zeros(*n, dtype=torch.complex128, device="cuda")
        d = lambda: torch.zeros(rhs, dtype=torch.float64, device="cuda")
        i = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
        self.m, self.rhs = m, rhs
        self.H, self.cs, self.sn = c(rhs, m, m + 1), c(rhs, m), c(rhs, m)  # H[r][column][row]
        self.g, self.y = c(rhs, m + 1), c(rhs, m)
        self.est, self.inv_h, self.abstol = d(), d(), d()
        self.active, self.any, self.kdone = i(rhs), i(1), i(rhs)
        self.host = torch.full((64,), -1, dtype=torch.int32, pin_memory=True)

    def arg(self):
        return State(*[getattr(self, k).data_ptr() for k, _ in State._fields_[:-1]], self.m)


def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1512_04506_amd as dd
    return dd.lib


T = {torch.complex64: "f", torch.complex128: "d"}


def stream():
    return vp(torch.cuda.current_stream().cuda_stream)


def start(K, V0, bo, cw, xo, yc, tol, nrhs):
    n, n_all = bo.shape[1], yc.shape[1]
    f = getattr(lib(), "_ZN5ddamg19launch_coarse_startI%sEEvNS_12ArnoldiStateEPNS_2cxIT_EEmPKS4_S7_mmS5_mS7_mmdPiii"
                       "P12ihipStream_t" % T[bo.dtype])
    f.argtypes = [State, vp, sz, vp, vp, sz, sz, vp, sz, vp, sz, sz, f64, vp, i32, i32, vp]
    f.restype = None
    f(K.arg(), V0.data_ptr(), n, bo.data_ptr(), cw.data_ptr() if cw is not None else None, n, n, xo.data_ptr(), n,
      yc.data_ptr(), n_all, n_all, tol, K.host.data_ptr(), nrhs, K.rhs, stream())
    torch.cuda.synchronize()


def fields(*shape, dtype=torch.complex64, seed=0):
    g = torch.Generator().manual_seed(seed)
    return torch.view_as_complex(torch.randn(*shape, 2, generator=g, dtype=torch.float64)).to(dtype).cuda()


def test_flags_left_by_a_call_of_more_rhs():
    """Six rhs active at the end of one solve (its iteration limit), two in the
    next: the count of active rhs is the new call's own, so that the gate of
    the operator shuts once those two have stopped."""
    n, K = 1000, Krylov(5, 8)
    bo, yc, x, V = (fields(8, k * n, seed=k) for k in (1, 2, 1, 1))
    start(K, V, bo, None, x, yc, -1.0, 6)
    assert K.active.tolist() == [1] * 6 + [0] * 2 and K.any.item() == 6 and K.host[:6].tolist() == [1] * 6
    start(K, V, bo, None, x, yc, -1.0, 2)
    assert K.active.tolist() == [1] * 2 + [0] * 6 and K.any.item() == 2
    start(K, V, bo, bo, x, yc, -1.0, 2)  # a later cycle whose residual is zero: both stop
    assert K.active.tolist() == [0] * 8 and K.any.item() == 0 and K.host[:2].tolist() == [0] * 2


def test_stop_threshold():
    """|y_c| of the longest vectors with one element per lane that swallows the
    squares added to it in FP32 (each below half its last bit): off by at most
    what a chain of 32 FP32 additions may lose, in the square 31 2^-24."""
    n, n_all, K = 24576, 49152, Krylov(3, 1)
    y = torch.full((1, n_all), (0.99 * 2.0 ** -24) ** 0.5, dtype=torch.complex64, device="cuda")
    y[0, :1024] = 1.0
    bo, x, V = (fields(1, n, seed=4) for _ in range(3))
    start(K, V, bo, None, x, y, 0.5, 1)
    want = 0.25 * float((y.to(torch.complex128).abs() ** 2).sum())
    assert abs(K.abstol.item() ** 2 / want - 1.0) <= 31 * 2.0 ** -24
