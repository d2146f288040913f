"""One FP32 layer X1 = a X0^2 + b X0 + c I of the tiled kernel (through fe_matrix_forward) against
FP64, at the smallest size, where K blocks and tiles leave remainders, and on either side of the size
where the tile grows from 32 to 64 (np 4096); arrays that start on 4 bytes only take the
element-wise loads and give the same bits.

Tolerance: a chain of n products and the three-term epilogue in FP32, u = 2^-24:
|fl - exact| <= (n + 4) u (|a| ||x_i|| ||x_j|| + |b x_ij| + |c| delta_ij)."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def layer(api, X0, theta, shift):
    n = X0.shape[0]
    buf = torch.zeros(2 * n * n + 8, dtype=torch.float32, device="cuda")
    out = torch.zeros(n * n + 8, dtype=torch.float32, device="cuda")
    buf[shift:shift + n * n] = X0.reshape(-1)
    th = np.ascontiguousarray(theta)
    api._check(api.lib().fe_matrix_forward(C.c_void_p(buf.data_ptr() + 4 * shift), n,
                                           th.ctypes.data_as(C.c_void_p), 1,
                                           C.c_void_p(out.data_ptr() + 4 * shift), api._stream_ptr()))
    torch.cuda.synchronize()
    return buf[shift + n * n:shift + 2 * n * n].reshape(n, n)


@pytest.mark.parametrize("n", [64, 192, 1024, 4096, 4160])
def test_one_layer(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    X = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g)
    X0 = (0.3 * (X + X.T) / n ** 0.5).float()
    X0.diagonal().add_(0.4)
    a, b, c = -1.3, 2.1, 0.05
    print(f"case n={n}", flush=True)
    X1 = layer(api, X0, [[a, b, c, 0.0]], 0)
    x = X0.double()
    ref = a * (x @ x) + b * x
    ref.diagonal().add_(c)
    r = torch.linalg.norm(x, dim=1)
    tol = abs(a) * r[:, None] * r[None, :] + abs(b) * x.abs()
    tol.diagonal().add_(abs(c))
    assert bool(((X1.double() - ref).abs() <= (n + 4) * 2.0 ** -24 * tol).all())
    assert torch.equal(X1, X1.T)
    assert torch.equal(layer(api, X0, [[a, b, c, 0.0]], 1), X1)


@pytest.mark.parametrize("n,shift", [(64, 0), (64, 1), (192, 0), (576, 0)])
def test_two_layer_backward(n, shift):
    """fe_matrix_backward against FP64 from the same states, for a G that is not symmetric. Layer 1's
    sums carry one product's rounding, layer 0's also that of the adjoint it starts from: with
    absolute values throughout, (n + 8) u and 3 (n + 8) u of the sums of magnitudes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_08523_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    rnd = lambda: torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g) / n ** 0.5  # noqa: E731
    sym = lambda m: (0.5 * (m + m.T)).float()  # noqa: E731
    X = [sym(rnd()), sym(rnd())]
    G = rnd().float()
    th = np.array([[-1.3, 2.1, 0.05, 0.4], [1.1, -0.3, 0.2, -0.7]])
    flat = torch.zeros(4 * n * n + 8, dtype=torch.float32, device="cuda")
    for k, m in enumerate(X + [G]):   # hist[0], hist[1]; G in the unused place of hist[2]
        flat[shift + k * n * n:shift + (k + 1) * n * n] = m.reshape(-1)
    work = torch.zeros(3 * n * n + 8, dtype=torch.float32, device="cuda")
    part = torch.full((4,), 7.0, dtype=torch.float64, device="cuda")
    grad = torch.zeros((2, 4), dtype=torch.float64, device="cuda")
    p = lambda t, o: C.c_void_p(t.data_ptr() + 4 * o)  # noqa: E731
    print(f"case n={n} shift={shift}", flush=True)
    api._check(api.lib().fe_matrix_backward(p(flat, shift), n, th.ctypes.data_as(C.c_void_p), 2,
                                            p(flat, shift + 2 * n * n), p(work, shift), p(part, 0), 1,
                                            p(grad, 0), api._stream_ptr()))
    torch.cuda.synchronize()
    Xd, Gd = [x.double() for x in X], G.double()

    def sums(Xb, x, gg, m):
        return torch.stack([(m * x).sum(), (Xb * x).sum(), Xb.diagonal().sum(), (gg * x).sum()])

    Xb, Ab = Gd, Gd.abs()
    for i in (1, 0):
        M, Mb = Xb @ Xd[i], Ab @ Xd[i].abs()
        tol = (1 if i else 3) * (n + 8) * 2.0 ** -24 * sums(Ab, Xd[i].abs(), Gd.abs(), Mb)
        assert bool(((grad[i] - sums(Xb, Xd[i], Gd, M)).abs() <= tol).all()), i
        a, b, _, d = th[i]
        Xb, Ab = a * (M + M.T) + b * Xb + d * Gd, abs(a) * (Mb + Mb.T) + abs(b) * Ab + abs(d) * Gd.abs()
    assert bool((part == 7.0).all())
