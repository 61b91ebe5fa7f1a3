"""CA-CFAR where the cheap FP32 sums may not decide: cells at and within
rounding of their threshold, values that are negative, not finite, denormal or
near the largest float, and rows around the ends of a 2048-cell tile.  The
mask equals the oracle's ordered FP64 one bit for bit."""
import numpy as np
import pytest

from oracle import cfar as ocfar
from tests.gpu_common import binding, dev, host

pytestmark = pytest.mark.gpu

P, S = 32, 2


def _rows(kind, R, n_ref, n_guard, alpha):
    rng = np.random.default_rng(R + n_ref)
    p = rng.exponential(1.0, (P, S, R)).astype(np.float32)
    if kind == "threshold":
        # every 97th cell moved to its own threshold, give or take an ulp
        n_used = 2 * n_ref
        for r in range(n_ref + n_guard, R - n_ref - n_guard, 97):
            w = np.concatenate([p[..., r - n_guard - n_ref:r - n_guard], p[..., r + n_guard + 1:r + n_guard + n_ref + 1]], -1)
            t = np.minimum(alpha * w.astype(np.float64).sum(-1) / n_used, 3e38).astype(np.float32)
            p[..., r] = np.where(np.arange(S) % 2, np.nextafter(t, np.float32(np.inf)), t)
    elif kind == "constant":
        p[:] = 1.5
    elif kind == "negative":
        p[..., ::301] *= -1
    elif kind == "not finite":
        p[0, 0, ::211], p[1, 1, ::211], p[2, :, ::211] = np.inf, np.nan, -np.inf
    elif kind == "denormal":
        p *= np.float32(1e-41)
    elif kind == "huge":
        p = np.minimum(p.astype(np.float64) * 3e37, 3.4e38).astype(np.float32)
    elif kind == "zero":
        p[:] = 0
        p[..., R // 2] = 1
    return p


@pytest.mark.parametrize("R,n_ref,n_guard", [(2048, 8, 0), (2049, 16, 2), (2047, 9, 3), (4100, 64, 64), (300, 31, 1)])
@pytest.mark.parametrize("kind", ["threshold", "constant", "negative", "not finite", "denormal", "huge", "zero"])
def test_cfar_mask_bitwise_at_the_margin(kind, R, n_ref, n_guard):
    stap = binding()
    for alpha in (1.0, ocfar.alpha_for_pfa(2 * n_ref, 1e-3), 1e-30, 1e30):
        p = _rows(kind, R, n_ref, n_guard, alpha)
        with np.errstate(invalid="ignore", over="ignore"):
            want, _, _ = ocfar.ca_cfar(p, n_ref, n_guard, alpha)
        got = host(stap.cfar(stap.problem(4, P, R, 3, 1, S), dev(p), n_ref, n_guard, alpha)).astype(bool)
        assert np.array_equal(got, want), (alpha, int((got != want).sum()))
