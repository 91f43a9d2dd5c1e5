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


def arnoldi(K, k, V, nrhs):
    n = V.shape[2]
    f = getattr(lib(), "_ZN5ddamg21launch_coarse_arnoldiI%sEEvNS_12ArnoldiStateEiPNS_2cxIT_EEmmmPiiP12ihipStream_t"
                % T[V.dtype])
    f.argtypes = [State, i32, vp, sz, sz, sz, vp, i32, vp]
    f.restype = None
    f(K.arg(), k, V.data_ptr(), V.shape[1] * n, n, n, K.host.data_ptr(), nrhs, stream())
    torch.cuda.synchronize()


def finish(K, V, xo, nrhs):
    n = V.shape[2]
    f = getattr(lib(), "_ZN5ddamg20launch_coarse_finishI%sEEvNS_12ArnoldiStateEPKNS_2cxIT_EEmmPS4_mmiP12ihipStream_t"
                % T[V.dtype])
    f.argtypes = [State, vp, sz, sz, vp, sz, sz, i32, vp]
    f.restype = None
    f(K.arg(), V.data_ptr(), V.shape[1] * n, n, xo.data_ptr(), n, n, nrhs, stream())
    torch.cuda.synchronize()


# one vector length for each number of elements per lane (4, 8, 16, 24 in FP32), whole and ragged
@pytest.mark.parametrize("n,steps,dtype", [(1000, 41, torch.complex64), (4096, 9, torch.complex128),
                                           (7001, 41, torch.complex64), (12288, 13, torch.complex64),
                                           (16384, 6, torch.complex128), (20480, 13, torch.complex64),
                                           (24576, 6, torch.complex64)])
def test_arnoldi_steps(n, steps, dtype):
    """A cycle with a diagonal operator: every new vector, column, rotation and
    estimate against the same step (classical Gram-Schmidt twice) in 64 bits on
    the device's own basis, past the groups of four vectors that a reduction
    and a back substitution take; the middle rhs never starts."""
    rhs, m = 3, 64
    eps = 2.0 ** (-24 if dtype == torch.complex64 else -53)
    K = Krylov(m, rhs)
    V = torch.zeros(steps + 1, rhs, n, dtype=dtype, device="cuda")
    A = fields(n, dtype=torch.complex128, seed=11)
    A = A / (1.0 + A.abs())  # entries of the unit disc
    bo, yc, x = (fields(rhs, n, dtype=dtype, seed=s) for s in (12, 13, 14))
    bo[1] = 0.0
    start(K, V[0], bo, None, x, yc, -1.0, rhs)
    assert K.active.tolist() == [1, 0, 1] and not bool(x.any())
    W = torch.complex128
    R = torch.zeros(rhs, m, m + 1, dtype=W, device="cuda")  # rotated columns
    rot = [[] for _ in range(rhs)]
    g = [[float(torch.linalg.vector_norm(bo[r].to(W)))] for r in range(rhs)]
    beta = [b[0] for b in g]
    small = 1.0
    for k in range(steps):
        w = (A * V[k].to(W)).to(dtype)
        w[1] = 7.0  # the idle rhs: left as it is
        V[k + 1] = w
        arnoldi(K, k, V, rhs)
        assert K.active.tolist() == [1, 0, 1] and K.any.item() == 2 and K.host[:3].tolist() == [1, 0, 1]
        assert K.inv_h[1].item() == 0.0 and bool((V[k + 1, 1] == 7.0).all())
        for r in (0, 2):
            B = V[:k + 1, r].to(W)
            v = w[r].to(W)
            h = torch.zeros(k + 1, dtype=W, device="cuda")
            for _ in range(2):
                d = B.conj() @ v
                h, v = h + d, v - B.T @ d
            hn, wn = float(torch.linalg.vector_norm(v)), float(torch.linalg.vector_norm(w[r].to(W)))
            small = min(small, hn / wn)
            tol = 16 * (k + 2) * eps / small
            assert float(torch.linalg.vector_norm(V[k + 1, r].to(W) - v / hn)) <= tol, (k, r)
            col = [complex(c) for c in h.tolist()] + [complex(hn)]
            for j, (c, s) in enumerate(rot[r]):
                col[j], col[j + 1] = c * col[j] + s * col[j + 1], c * col[j + 1] - s.conjugate() * col[j]
            a, b = col[k], col[k + 1]
            nrm = (abs(a) ** 2 + abs(b) ** 2) ** 0.5
            c, s = abs(a) / nrm, (a / abs(a)) * b.conjugate() / nrm
            rot[r].append((c, s))
            col[k], col[k + 1] = nrm * a / abs(a), 0.0
            gk = g[r][k]
            g[r][k:] = [c * gk, -s.conjugate() * gk]
            R[r, k, :k + 2] = torch.tensor(col, dtype=W)
            tol = 64 * (k + 2) * eps / small
            assert float((K.H[r, k, :k + 2] - R[r, k, :k + 2]).abs().max()) <= tol * wn, (k, r)
            assert abs(K.est[r].item() - abs(g[r][k + 1])) <= tol * beta[r], (k, r)
    # the end of the cycle from the device's own triangle and right-hand side
    x0 = fields(rhs, n, dtype=dtype, seed=15)
    x = x0.clone()
    finish(K, V, x, rhs)
    assert K.kdone.tolist() == [steps, 0, steps] and torch.equal(x[1], x0[1])
    for r in (0, 2):
        tri = K.H[r, :steps, :steps].T.contiguous()
        y = torch.linalg.solve_triangular(tri, K.g[r, :steps, None], upper=True)[:, 0]
        want = x0[r].to(W) + V[:steps, r].to(W).T @ y
        scale = float(torch.linalg.vector_norm(x0[r].to(W))) + float(y.abs().sum())
        assert float(torch.linalg.vector_norm(x[r].to(W) - want)) <= 4 * (steps + 2) * eps * scale


@pytest.mark.parametrize("restart", (6, 30))
@pytest.mark.parametrize("L,ntv", [((8, 8, 8, 8), 24), ((8, 8, 8, 16), 24), ((8, 8, 16, 16), 20)])
def test_vcycle_past_four_columns(L, ntv, restart):
    """Nine coarse iterations, over a restart and in one cycle, on vectors of
    6144, 12288 (steps beyond the fourth take many workgroups) and 20480
    elements (FP64: many throughout) against FP64."""
    lib()
    import paper_1512_04506_amd as dd
    import synth
    U = torch.from_numpy(synth.su3_field(L, 0.4, 941)).cuda()
    tv = torch.from_numpy(synth.gaussian_spinors(L, ntv, 942)).cuda()
    y = torch.from_numpy(synth.gaussian_spinors(L, 2, 943)).cuda()
    xs = []
    for prec in (dd.FP64, dd.FP32, dd.MIXED16):
        ctx = dd.Context(dd.default_params(L=L, block=(2, 2, 2, 2), m0=-0.1, ntv=ntv, prec=prec, max_rhs=2,
                                           coarse_restart=restart, coarse_fixed_its=9), U)
        ctx.import_tv(tv)
        x = torch.empty_like(y)
        for _ in range(3):  # replays of the captured steps among them
            ctx.mg_apply(x, y, 2)
        xs.append(x)
        ctx.close()
    for x, tol in ((xs[1], 1e-5), (xs[2], 1e-2)):  # the parity bars of the V-cycle
        assert float((x - xs[0]).abs().max() / xs[0].abs().max()) <= tol
