"""GPU parity of the inner products at the edges of their dispatch: one, two,
four and eight waves per system (by block length, DOF and steering vectors),
full and ragged tiles of range cells, DOF and steering vectors, on the plain
and the mixed path.  Element by element against the FP64 products of the same
inputs: |error of y| <= 4 (D + 4) u sum |w| |x|, as for a covariance element
over D terms."""
import numpy as np
import pytest

from tests.gpu_common import U32, binding, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 16, 17, 32, 33, 64, 65, 100])
@pytest.mark.parametrize("C,T,S", [(4, 3, 8), (11, 3, 17), (16, 4, 33), (24, 4, 16), (32, 4, 64), (43, 3, 32),
                                   (64, 3, 49), (64, 3, 64)], ids=str)
def test_inner_products_edges(C, T, S, N):
    stap = binding()
    P, B, D = 32, 3, C * T
    rng = np.random.default_rng(1000 * D + 10 * S + N)
    cplx = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    X, W = cplx(P, D, B * N), cplx(P, B, S, D)
    X *= np.float32(10.0) ** rng.integers(-3, 4, (P, D, 1)).astype(np.float32)
    Xb = X.astype(np.complex128).reshape(P, D, B, N).transpose(0, 2, 1, 3)
    want = np.matmul(W.astype(np.complex128).conj(), Xb).transpose(0, 2, 1, 3).reshape(P, S, B * N)
    size = np.matmul(np.abs(W), np.abs(Xb)).transpose(0, 2, 1, 3).reshape(P, S, B * N)
    got = []
    for precision in ("fp32", "bf16"):
        p, y = stap.inner_products(stap.problem(C, P, B * N, T, B, S, precision=precision), dev(W), dev(X), want_y=True)
        p, y = host(p), host(y)
        assert np.all(np.abs(y - want) <= 4.0 * (D + 4) * U32 * size)
        y64 = y.astype(np.complex128)
        assert np.allclose(p, np.abs(y64) ** 2, rtol=4 * U32, atol=0)
        got.append((p, y))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
