"""With refinement no route of stap_run keeps a covariance in the workspace up
to 128 DOF: it is not asked for, and the cubes that fit the no-allocation entry
point without it run there."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_common import dev, host, prob_of


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("C,S,R,B", [(4, 8, 512, 32), (16, 16, 1000, 10), (32, 32, 256, 2), (40, 20, 256, 2)])
def test_refined_workspace_has_no_covariance(C, S, R, B, precision):
    from paper_2203_06233_amd import stap
    P, D = 32, 3 * C
    up = lambda n: (n + 255) // 256 * 256
    plain, refined = (stap.workspace_size([stap.problem(C, P, R, 3, B, S, precision=precision, refine_steps=r)])
                      for r in (0, 1))
    parts = up(P * D * R * 8) + up(P * B * S * D * 8) + up(P * B * 4)
    cov = up(P * B * D * D * 8) + up(P * B * 4)
    assert refined - parts == plain - parts - (cov if D <= 96 else 0) and refined - parts <= 1024


@pytest.mark.gpu
def test_refined_cube_fits_the_fixed_scratch():
    from paper_2203_06233_amd import stap
    wl = synth.Workload("scratch", 16, 64, 4096, 3, 256, 16, cnr_db=30.0, seed=2)
    prob = prob_of(wl, "bf16", 1)
    assert stap.workspace_size([prob]) <= stap.NOALLOC_MAX_BYTES
    cube, V = dev(synth.make_cube(wl)), dev(synth.steering(wl))
    power = torch.empty((wl.n_pulse, wl.n_steer, wl.n_range), dtype=torch.float32, device="cuda")
    stap.run_noalloc([prob], [cube], [V], [power])
    assert np.array_equal(host(power), host(stap.run([prob], [cube], [V])[0]))
