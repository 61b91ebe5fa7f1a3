"""The refined solve of shape classes that nobody tuned takes the blocked
matrix-core kernel.  Its weights are held to those of the column sweep, whose
arithmetic is FP32 throughout: no further from the 64-bit ones than the sweep
is with as many refinement steps, or than the roundings that end every solve
(u_s 1, gamma 1/2, square root 2, reciprocal 1, product 1 unit and a half to
spare: 6 units), on clutter covariances of condition 1e4 to 1e6."""
import numpy as np
import pytest

import synth
from oracle import metrics
from oracle import stap as orc
from tests.gpu_common import U32, binding, dev, host, prob_of
from tests.test_gpu_parity import solve_variant

pytestmark = pytest.mark.gpu

# (C, T, S) off the tuned classes, at the edges of their block columns
SHAPES = [(5, 3, 24), (8, 3, 40), (11, 3, 40), (16, 3, 33), (49, 1, 16), (17, 3, 40), (16, 4, 8), (28, 3, 48), (32, 3, 64),
          (33, 3, 16), (40, 3, 20), (32, 4, 64), (43, 3, 16), (64, 3, 31)]


@pytest.mark.parametrize("eps", [1e-3, 1e-4])
@pytest.mark.parametrize("kind,precision", [(0, "fp32"), (0, "bf16"), (1, "fp32")])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_refined_weights_as_close_as_the_column_sweep(shape, kind, precision, eps):
    stap = binding()
    C, T, S = shape
    D, P, B = C * T, 32, 2
    if kind == 0 and D > 128:
        pytest.skip("the fused kernels end at 128 DOF")
    assert stap.tune_get(D, S, precision, 1, kind=kind) == 0  # the default is what is tested
    wl = synth.with_(synth.Workload("default", C, P, 2 * D * B, T, B, S, cnr_db=40.0, seed=5), load_eps=eps)
    X = dev(orc.doppler(synth.make_cube(wl), T).astype(np.complex64))
    V = synth.steering(wl)
    prob = prob_of(wl, precision, 1)
    cov = stap.covariance(prob, X)[0]
    want, _, _ = orc.solve_weights(host(cov).astype(np.complex128), V)

    def error():
        w, info = stap.covariance_solve(prob, X, dev(V)) if kind == 0 else stap.solve_weights(prob, cov, dev(V))
        assert np.all(host(info) == 0)
        return metrics.per_system_rel_err(host(w), want)

    got = error()
    with solve_variant(stap, kind, D, S, precision, 1, 16):
        sweep = error()
    print("refined", shape, kind, precision, eps, float(got.max()), float(sweep.max()), flush=True)
    assert np.all(got <= np.maximum(sweep.max(), 6 * U32))


@pytest.mark.parametrize("steps", [2, 4])
@pytest.mark.parametrize("shape", [(5, 3, 24), (10, 3, 50), (16, 3, 33), (17, 3, 40), (32, 3, 64), (40, 3, 20), (64, 3, 16)],
                         ids=str)
def test_more_steps_and_one_cube_as_in_a_batch(shape, steps):
    """Several requested steps on the default route, by stage and fused, and
    two cubes of the class in one call with the bits they have alone."""
    stap = binding()
    C, T, S = shape
    D, P, B = C * T, 32, 2
    wl = synth.Workload("steps", C, P, 2 * D * B, T, B, S, cnr_db=40.0, seed=6)
    cube, V = dev(synth.make_cube(wl)), dev(synth.steering(wl))
    prob = prob_of(wl, "fp32", steps)
    X = stap.doppler(prob, cube)
    cov = stap.covariance(prob, X)[0]
    want, _, _ = orc.solve_weights(host(cov).astype(np.complex128), synth.steering(wl))
    w, info = stap.solve_weights(prob, cov, V)
    assert np.all(host(info) == 0) and metrics.per_system_rel_err(host(w), want).max() <= 6 * U32
    if D <= 128:
        w, info = stap.covariance_solve(prob, X, V)
        assert np.all(host(info) == 0) and metrics.per_system_rel_err(host(w), want).max() <= 6 * U32
    one = host(stap.run([prob], [cube], [V])[0])
    for p in stap.run([prob] * 2, [cube] * 2, [V] * 2):
        assert np.array_equal(host(p), one)
