"""stap_solve_weights reads the lower triangle of the covariance alone: with
NaN in the strict upper triangle and in the imaginary part of the diagonal
every solve gives the bits it gives for the full Hermitian matrix."""
import numpy as np
import pytest

import synth
from oracle import stap as orc
from tests.gpu_common import binding, dev, host, prob_of
from tests.test_gpu_parity import solve_variant

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("refine", [0, 1])
@pytest.mark.parametrize("variant", [0, 1, 4, 8, 16, 32])
@pytest.mark.parametrize("shape", [(4, 3, 8), (17, 1, 20), (13, 3, 11), (16, 4, 32), (27, 3, 17), (32, 3, 32),
                                   (40, 3, 20)], ids=str)
def test_solve_reads_the_lower_triangle_alone(shape, variant, refine):
    stap = binding()
    C, T, S = shape
    D, P, B = C * T, 32, 2
    wl = synth.Workload("lower", C, P, 2 * D * B, T, B, S, cnr_db=30.0, seed=9)
    prob = prob_of(wl, "fp32", refine)
    X = dev(orc.doppler(synth.make_cube(wl), T).astype(np.complex64))
    cov, V = host(stap.covariance(prob, X)[0]), dev(synth.steering(wl))
    lower = np.tril(cov)
    nan = np.float32(np.nan)
    i, j = np.triu_indices(D, 1)
    lower[..., i, j] = nan + 1j * nan
    lower.imag[..., np.arange(D), np.arange(D)] = nan
    with solve_variant(stap, 1, D, S, "fp32", refine, variant):
        want = [host(x) for x in stap.solve_weights(prob, dev(cov), V)]
        got = [host(x) for x in stap.solve_weights(prob, dev(lower), V)]
    assert np.all(want[1] == 0) and np.all(np.isfinite(want[0]))
    assert np.array_equal(got[1], want[1]) and np.array_equal(got[0], want[0])
