"""Inner products of values that three BF16 terms do not hold: infinite and
NaN samples and weights, finite ones that round to infinity in BF16, and data
or weights so small that the lower terms are denormal.  The results are those
of FP32 products: the 64-bit ones within 4 (D + 4) u sum |w| |x| wherever
those are finite, an infinite power where a sample or a weight is infinite,
NaN where one is NaN, and nothing beside them changes.  The mixed path up to 128 DOF
has the split alone and is not held to this."""
import numpy as np
import pytest

from tests.gpu_common import U32, binding, dev, host

pytestmark = pytest.mark.gpu

P, B = 32, 2


def _data(D, S, N, seed):
    rng = np.random.default_rng(seed)
    cplx = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    return cplx(P, D, B * N), cplx(P, B, S, D)


def _products(X, W, N):
    Xb = X.astype(np.complex128).reshape(P, -1, B, N).transpose(0, 2, 1, 3)
    y = lambda w, x: np.matmul(w, x).transpose(0, 2, 1, 3).reshape(P, W.shape[2], B * N)
    return y(W.astype(np.complex128).conj(), Xb), y(np.abs(W.astype(np.complex128)), np.abs(Xb))


@pytest.mark.parametrize("precision", ["fp32", "fp8"])
@pytest.mark.parametrize("C,T,S,N", [(4, 3, 8, 16), (4, 3, 40, 100), (13, 3, 11, 33), (32, 3, 32, 128), (43, 3, 17, 24),
                                     (64, 3, 64, 80)], ids=str)
@pytest.mark.parametrize("what", ["inf", "big", "nan", "tiny cells", "tiny data", "tiny weights", "inf weight"])
def test_inner_products_out_of_the_split_s_range(what, C, T, S, N, precision):
    stap = binding()
    if C * T <= 128 and precision == "fp8":
        pytest.skip("the split alone")
    D = C * T
    X, W = _data(D, S, N, 7 * D + S)
    cells = np.zeros(B * N, bool)   # cells (or, for a weight, blocks) whose products are not finite
    bad = slice(0, 0)
    if what in ("inf", "nan"):
        X[:, D // 2, 5] = np.inf if what == "inf" else np.nan
        cells[5] = True
    elif what == "big":
        X[:, D // 2, 5] = 3.4e38
        W *= np.float32(1e-3)
    elif what == "tiny cells":
        X[:, :, N:N + 3] *= np.float32(1e-36)
    elif what == "tiny data":
        X *= np.float32(1e-36)
        W *= np.float32(1e20)
    elif what == "tiny weights":
        W[:, 1, S // 2] *= np.float32(1e-36)
        X *= np.float32(1e20)
    else:
        W[:, 0, S - 1, 1] = np.inf
        bad, cells[:N] = slice(S - 1, S), True
    p, y = stap.inner_products(stap.problem(C, P, B * N, T, B, S, precision=precision), dev(W), dev(X), want_y=True)
    p, y = host(p), host(y)
    rows = np.zeros((P, S, B * N), bool)
    if bad != slice(0, 0):
        rows[:, bad, :N] = True
    else:
        rows[..., cells] = True
    with np.errstate(all="ignore"):
        want, size = _products(X, W, N)
        y64 = y.astype(np.complex128)
        # FP32's own smallest step is all that a result below 2^-126 can keep
        assert np.all(np.abs(y64 - want)[~rows] <= (4.0 * (D + 4) * U32 * size)[~rows] + D * 2.0 ** -148)
        power = (np.abs(y64) ** 2)[~rows]
        assert np.allclose(p[~rows], np.where(power > 3.4e38, np.inf, power), rtol=4 * U32, atol=2.0 ** -148)
    if rows.any():
        assert np.all(np.isnan(p[rows]) if what == "nan" else np.isinf(p[rows]))
