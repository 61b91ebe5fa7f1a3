"""GPU parity of the Doppler tiles of large launches (wide tiles, tiles dealt
to the XCDs in runs), element by element: range cells that are no multiple of
a tile, numbers of tiles that are no multiple of eight, each tap count, both
tap phases, subarrays and pulses outermost; and cubes that reach those tiles
only together, whose results are the bits they have alone."""
import numpy as np
import pytest

import synth
from oracle import stap as orc
from tests.gpu_common import binding, dev, fft_bound, host, prob_of

pytestmark = pytest.mark.gpu

# (C, P, R, T, n_sub): C channels; 512 tiles of 32 cells (256, 512 pulses) or of
# 64 (128), 256 of 128 (64) or 274 of 96 (100) take the wide shape
WIDE = [(43, 64, 770, 2, 1), (37, 64, 1025, 4, 1), (43, 100, 650, 3, 1), (23, 100, 1250, 2, 3), (29, 100, 1000, 1, 8),
        (43, 128, 781, 1, 1), (43, 128, 769, 3, 1), (37, 256, 433, 2, 1), (41, 256, 417, 4, 1), (37, 512, 433, 2, 1),
        (33, 512, 511, 3, 1)]


@pytest.mark.parametrize("outer", [False, True], ids=["", "pulse-outer"])
@pytest.mark.parametrize("phase", ["absolute", "relative"])
@pytest.mark.parametrize("shape", WIDE, ids=str)
def test_doppler_wide_tiles(shape, phase, outer):
    stap = binding()
    C, P, R, T, n_sub = shape
    rng = np.random.default_rng(C + P + R)
    cube = (rng.standard_normal((C * n_sub, P, R)) + 1j * rng.standard_normal((C * n_sub, P, R))).astype(np.complex64)
    kw = dict(cube_stride_chan=R, cube_stride_pulse=C * n_sub * R) if outer else {}
    prob = stap.problem(C * n_sub, P, R, T, 1, 1, tap_phase=phase, n_sub=n_sub, **kw)
    X = host(stap.doppler(prob, dev(np.ascontiguousarray(cube.transpose(1, 0, 2)) if outer else cube)))
    summed = cube.astype(np.complex128).reshape(C, n_sub, P, R).sum(1)
    want = orc.doppler(summed, T)
    if phase == "relative":
        k, t = np.arange(P)[:, None], np.repeat(np.arange(T), C)[None, :]
        want = want * np.exp(2j * np.pi * (k * t % P) / P)[..., None]
    size = np.abs(cube).reshape(C, n_sub, P, R).sum(1)  # the sum of a subarray's elements rounds too
    assert np.all(np.abs(X - want) <= fft_bound(size, T, c=8.0 + n_sub - 1))


@pytest.mark.parametrize("P,cubes", [(64, [(16, 700, 1), (13, 900, 1), (16, 800, 1)]), (128, [(16, 700, 1), (13, 900, 1), (16, 800, 1)]),
                                     (256, [(16, 330, 1), (13, 450, 1), (16, 400, 1)]), (512, [(16, 330, 1), (13, 450, 1), (16, 400, 1)]),
                                     (100, [(16, 600, 1), (13, 900, 2), (16, 700, 1)])], ids=str)
def test_cubes_that_are_wide_together(P, cubes):
    stap = binding()
    wls = [synth.Workload(f"w{i}", C * sub, P, R, 3, R // 50, 8, cnr_db=30.0, seed=3 + i, n_sub=sub)
           for i, (C, R, sub) in enumerate(cubes)]
    probs = [prob_of(w, "fp32", 0) for w in wls]
    xs, vs = [dev(synth.make_cube(w)) for w in wls], [dev(synth.steering(w)) for w in wls]
    both = [host(p) for p in stap.run(probs, xs, vs)]
    for i, one in enumerate(probs):
        X = stap.doppler(one, xs[i])
        w, info = stap.covariance_solve(one, X, vs[i])
        assert np.all(host(info) == 0)
        assert np.array_equal(both[i], host(stap.inner_products(one, w, X))), i


@pytest.mark.parametrize("outer", [False, True], ids=["", "pulse-outer"])
@pytest.mark.parametrize("n_sub", [2, 3, 4, 5, 8, 11])
@pytest.mark.parametrize("shape", [(3, 32, 130, 2), (2, 64, 95, 3), (5, 32, 33, 1), (2, 128, 40, 1)], ids=str)
def test_subarrays_on_narrow_tiles(shape, n_sub, outer):
    """Elements read four at a time (32 and 64 pulses), with and without a remainder."""
    test_doppler_wide_tiles((*shape, n_sub), "absolute", outer)
