"""The refined blocked solve does not depend on the scale of the data:
covariances from 2^-80 to 2^124 give the weights of the unscaled system times
the matching power of two, bit for bit, and down to 2^-108, where FP32 itself
drops bits of the smallest elements, the accuracy of the unscaled system."""
import numpy as np
import pytest

import synth
from oracle import metrics
from oracle import stap as orc
from tests.gpu_common import U32, binding, dev, host, prob_of
from tests.test_gpu_parity import solve_variant

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 8])
@pytest.mark.parametrize("shape", [(16, 4, 8), (32, 3, 64), (40, 3, 20), (64, 3, 31)], ids=str)
def test_refined_weights_at_any_scale(shape, variant):
    stap = binding()
    C, T, S = shape
    D, P, B = C * T, 32, 2
    wl = synth.Workload("scaled", C, P, 2 * D * B, T, B, S, cnr_db=30.0, seed=5)
    X = dev(orc.doppler(synth.make_cube(wl), T).astype(np.complex64))
    V = synth.steering(wl)
    prob = prob_of(wl, "fp32", 1)
    cov = host(stap.covariance(prob, X)[0])
    top = int(np.floor(np.log2(np.abs(cov).max())))
    w = {}
    with solve_variant(stap, 1, D, S, "fp32", 1, variant):
        for size in (None, -108, -80, 108, 124):
            e = 0 if size is None else (size - top) & ~1  # a power of four
            scaled = cov * np.float32(2.0 ** (e // 2)) * np.float32(2.0 ** (e - e // 2))
            got, info = stap.solve_weights(prob, dev(scaled), dev(V))
            assert np.all(host(info) == 0), size
            w[size] = host(got).astype(np.complex128) * 2.0 ** (e // 2)
            if variant == 0:  # the corrected form, converged to its last roundings
                want, _, _ = orc.solve_weights(scaled.astype(np.complex128), V)
                assert metrics.per_system_rel_err(host(got), want).max() <= 6 * U32, size
    for size in (-80, 108, 124):
        assert np.array_equal(w[size], w[None]), size
