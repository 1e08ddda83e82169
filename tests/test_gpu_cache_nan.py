"""Proposed angles that are not finite, in the direct sweeps' seeded search on the
crown problem with the Euler foot: such a control's foot lies outside the domain
(value M), wherever the cell of the coast foot is.  So the node coasts, with the
value of a frozen-policy coast sweep bit for bit, and where the fallback
test asks for the full search its result is that of the scan + golden sweep.
The nodes in question are those on the lowest v_r and v_t faces, onto which a
clamp would put the foot; values fall towards them."""
import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [float("nan"), float("inf"), -float("inf")])
def test_seed_without_a_number_is_outside_the_domain(seed):
    from paper_2407_14675_amd import dpo

    p = inputs.crown_problem((12, 7, 9, 8), integrator="euler")
    p["search"] = dict(inputs.SEEDED, fallback_tol=1e9)
    print("seed", seed, flush=True)
    ctx = dpo.Context(p)
    n = p["n"]
    k = np.arange(n[2])[:, None, None] + np.arange(n[1])[None, :, None] + 0 * np.arange(n[0])[None, None, :]
    V = inputs.random_value(p, seed=73, high=0.5) + 10.0 * k[None]
    V = torch.from_numpy(np.ascontiguousarray(V, np.float32)).cuda()
    W, coast = V.clone(), V.clone()
    ang, thr = ctx.empty_policy()
    bad = torch.full_like(V, seed)
    ctx.bellman_sweep_seeded(V, W, ang, thr, bad)
    ctx.policy_eval_sweep(V, coast, torch.zeros_like(V), torch.zeros_like(thr))
    torch.cuda.synchronize()
    assert int(thr.sum()) == 0
    np.testing.assert_array_equal(W.cpu().numpy(), coast.cpu().numpy())
    # every node's value moves: all of them repeat the full search
    ctx.set_search(dict(inputs.SEEDED, fallback_tol=0.0))
    got = [V.clone(), *ctx.empty_policy()]
    want = [V.clone(), *ctx.empty_policy()]
    ctx.bellman_sweep_seeded(V, *got, bad)
    ctx.set_search(inputs.SCAN_GOLDEN)
    ctx.bellman_sweep(V, *want)
    torch.cuda.synchronize()
    assert bool((coast != V).all())
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
