"""The direct Heun sweep on both sides of the size where it changes from keyed
corners to the cell cache (327,680 free nodes), against frozen-policy sweeps
of every single control; odd sides put a row of nodes on v_r = 0 and on the
circular speed, whose feet hover about a face."""
import math

import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu

K = 6


@pytest.mark.parametrize("n", [(40, 19, 21, 20), (40, 20, 20, 20), (41, 21, 20, 20), (64, 16, 16, 20)])
def test_heun_sweep_is_the_least_single_control(n):
    from paper_2407_14675_amd import dpo

    p = inputs.crown_problem(n, n_angles=K)
    print("keyed corners", n, flush=True)
    ctx = dpo.Context(p)
    V = torch.from_numpy(inputs.random_value(p, seed=72, high=30.0)).float().cuda()
    W = V.clone()
    ang, thr = ctx.empty_policy()
    ctx.bellman_sweep(V, W, ang, thr)
    best, one = V.clone(), torch.zeros_like(V)
    ctx.policy_eval_sweep(V, best, ang, torch.zeros_like(thr))
    for k in range(K):
        u = np.float32(-math.pi + 2.0 * math.pi * k / K)
        ctx.policy_eval_sweep(V, one, torch.full_like(V, float(u)), torch.ones_like(thr))
        best = torch.minimum(best, one)
    torch.cuda.synchronize()
    d = (W - best).abs().cpu().numpy()
    # a foot known to 1e-6 cell along four axes, a slope of at most 30 per cell,
    # and one unit in the last place of values up to 60 and their running cost
    bound = 4 * 30.0 * 1e-6 + 2.0**-23 * np.maximum(best.abs().cpu().numpy(), 60.0) * 4
    # feet within rounding of the domain's r faces may part (M = 1e6 outside)
    assert np.mean(d > bound) < 1e-3
