"""The direct sweeps with the Heun foot, on the crown and the orbit problem and with
either form of the cell's cache, against frozen-policy sweeps of every single
control: every node whose feet all keep a distance from the domain's faces, in
FP64, meets the bound.  And the crown's scan + golden search with the Euler foot:
its value is its policy's own evaluation and no larger than the best sample's."""
import math

import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu

# a foot known to 1e-6 cell along four axes, a slope of at most 30 per cell, and one
# unit in the last place of values up to 60 and their running cost
SLOPE, NEAR = 30.0, 1e-5


def bound(v):
    return 4 * SLOPE * 1e-6 + 2.0**-23 * np.maximum(np.abs(v), 60.0) * 4


def near_a_face(p, K):
    """Nodes with a foot (coast or one of K angles) within NEAR cells of a face that is an
    exit: along r on the crown problem, along every axis on the orbit problem."""
    n, crown, dt = p["n"], p["model"] == "crown", p["dt"]
    h = [(p["hi"][k] - p["lo"][k]) / (n[k] if crown and k == 3 else n[k] - 1) for k in range(4)]
    axis = [(p["lo"][k] + np.arange(n[k]) * h[k]).reshape([-1 if 3 - q == k else 1 for q in range(4)]) for k in range(4)]
    x = np.broadcast_arrays(*axis)

    def slope(x, thr, u):
        r, vr, vt, w = x
        a = thr * p["accel"] / (1.0 if crown else w)
        return [vr, vt * vt / r - p["mu"] / r**2 + a * math.sin(u), -vr * vt / r + a * math.cos(u),
                vt / r if crown else -p["mdot"] * thr + 0.0 * r]

    near = np.zeros(x[0].shape, bool)
    for thr, u in [(0.0, 0.0)] + [(1.0, -math.pi + 2 * math.pi * k / K) for k in range(K)]:
        b = slope(x, thr, u)
        c = slope([x[k] + dt * b[k] for k in range(4)], thr, u)
        for k in (0,) if crown else range(4):
            s = (x[k] - p["lo"][k] + 0.5 * dt * (b[k] + c[k])) / h[k]
            near |= (np.abs(s) < NEAR) | (np.abs(s - (n[k] - 1)) < NEAR)
    return near


def least(ctx, V, K):
    ang, thr = ctx.empty_policy()
    best, one = V.clone(), torch.zeros_like(V)
    ctx.policy_eval_sweep(V, best, ang, torch.zeros_like(thr))
    for k in range(K):
        u = np.float32(-math.pi + 2.0 * math.pi * k / K)
        ctx.policy_eval_sweep(V, one, torch.full_like(V, float(u)), torch.ones_like(thr))
        best = torch.minimum(best, one)
    return best


@pytest.mark.parametrize("model,n,K", [("crown", (12, 7, 9, 8), 24), ("crown", (40, 19, 21, 20), 24),
                                       ("crown", (64, 17, 18, 18), 40), ("orbit", (12, 13, 11, 9), 24),
                                       ("orbit", (31, 23, 22, 22), 40)])
def test_heun_sweep_is_the_least_single_control(model, n, K):
    from paper_2407_14675_amd import dpo

    table = dict(mode="table", n_angles=K)
    p = inputs.crown_problem(n, n_angles=K) if model == "crown" else dict(inputs.orbit_problem(n, search=table), integrator="heun")
    print("heun controls", model, n, flush=True)
    ctx = dpo.Context(p)
    V = torch.from_numpy(inputs.random_value(p, seed=72, high=SLOPE)).float().cuda()
    W = V.clone()
    ctx.bellman_sweep(V, W, *ctx.empty_policy())
    best = least(ctx, V, K)
    torch.cuda.synchronize()
    check = (ctx.kind().cpu().numpy() == 0) & ~near_a_face(p, K)
    assert check.mean() > 0.5
    W, best = W.cpu().numpy()[check], best.cpu().numpy()[check]
    assert np.all(np.abs(W - best) <= bound(best))


@pytest.mark.parametrize("n", [(12, 7, 9, 8), (40, 20, 20, 20)])
def test_crown_scan_golden_value_is_its_policys(n):
    from paper_2407_14675_amd import dpo

    p = inputs.crown_problem(n, integrator="euler")
    p["search"] = dict(inputs.SCAN_GOLDEN)
    print("crown scan + golden", n, flush=True)
    ctx = dpo.Context(p)
    V = torch.from_numpy(inputs.random_value(p, seed=73, high=SLOPE)).float().cuda()
    W, own = V.clone(), V.clone()
    ang, thr = ctx.empty_policy()
    ctx.bellman_sweep(V, W, ang, thr)
    ctx.policy_eval_sweep(V, own, ang, thr)
    best = least(ctx, V, inputs.SCAN_GOLDEN["n_scan"])
    torch.cuda.synchronize()
    W, own, best = (t.cpu().numpy() for t in (W, own, best))
    assert np.all(np.abs(W - own) <= bound(own))
    # the golden section gains at most slope x step x (1 - cos(pi / 64)), here less than the bound
    assert np.all(W <= best + bound(best)) and (W < best).any()
