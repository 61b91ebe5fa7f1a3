"""GPU parity of the fused covariance->blocked solve at the edges of its block
layouts: one to eight block columns and one to four steering blocks, full and
ragged, on one, two, four and eight waves per system, without refinement
(FP32 products) and with one and two steps (split-BF16 products, the current
solution parked in LDS and in the weights array).

The covariance is the stage kernel's, which the fused kernel forms tile by
tile with the same arithmetic, so the oracle solves the very matrix the kernel
factors.  Bounds as for the stage solves: 8 D cond(R_L) u on the weights,
8 D u on the backward error.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import metrics
from oracle import stap as orc
from tests.gpu_common import U32, binding, dev, host, prob_of
from tests.test_gpu_parity import solve_variant

pytestmark = pytest.mark.gpu

# (C, T, S): D = C T and S at, below and above multiples of 16
EDGES = [(16, 1, 1), (5, 3, 16), (17, 1, 17), (8, 4, 32), (11, 3, 33), (16, 3, 16), (49, 1, 20), (16, 4, 64),
         (65, 1, 16), (24, 3, 31), (32, 3, 32), (32, 3, 64), (97, 1, 17), (32, 4, 16), (32, 4, 64)]


@pytest.mark.parametrize("refine", [0, 1, 2])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("edge", EDGES, ids=str)
def test_fused_blocked_solve_edges(edge, precision, refine):
    stap = binding()
    C, T, S = edge
    D, P, B = C * T, 32, 3
    N = 2 * D + 5
    wl = synth.Workload(f"edge-{C}-{T}-{S}", C, P, N * B, T, B, S, cnr_db=30.0, seed=21)
    X = dev(orc.doppler(synth.make_cube(wl), T).astype(np.complex64))
    V = synth.steering(wl)
    prob = prob_of(wl, precision, refine)
    R = host(stap.covariance(prob, X)[0]).astype(np.complex128)
    w0 = torch.full((P, B, S, D), complex(np.nan, np.nan), dtype=torch.complex64, device="cuda")
    i0 = torch.full((P, B), -7777, dtype=torch.int32, device="cuda")
    with solve_variant(stap, 0, D, S, precision, refine, 8):
        w, info = stap.covariance_solve(prob, X, dev(V), w=w0, info=i0)
    w, info = host(w), host(info)
    assert np.all(info == 0) and np.all(np.isfinite(w))
    Wo, _, _ = orc.solve_weights(R, V)
    bound = 8.0 * D * np.linalg.cond(R) * U32
    assert np.all(metrics.per_system_rel_err(w, Wo) <= bound)
    # backward error, the solution recovered from w: gamma = (v^H w)^2, u = w v^H w
    w = w.astype(np.complex128)
    u = w * np.real(np.sum(np.conj(V.astype(np.complex128)) * w, axis=-1))[..., None]
    res = np.einsum("kbij,kbsj->kbsi", R, u) - V
    scale = np.linalg.norm(R, 2, axis=(-2, -1))[..., None] * np.linalg.norm(u, axis=-1)
    assert np.all(np.linalg.norm(res, axis=-1) <= 8.0 * D * U32 * scale)


@pytest.mark.parametrize("shape", [(4, 8), (8, 24), (13, 11), (20, 33), (32, 32)], ids=str)
def test_one_cube_and_batch_agree_with_refinement(shape):
    """One cube alone and in a batch of its shape class take different
    launches (and may take different wave counts); the bits are the same."""
    stap = binding()
    C, S = shape
    wls = [synth.Workload(f"pair{i}", C, 32, 64 * (3 + i), 3, 3 + i, S, cnr_db=40.0, seed=31 + i) for i in range(2)]
    cubes, Vs = [dev(synth.make_cube(w)) for w in wls], [dev(synth.steering(w)) for w in wls]
    probs = [prob_of(w, "bf16", 1) for w in wls]
    both = [host(p) for p in stap.run(probs, cubes, Vs)]
    for i in range(2):
        assert np.array_equal(both[i], host(stap.run([probs[i]], [cubes[i]], [Vs[i]])[0])), i
