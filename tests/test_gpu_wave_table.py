"""The closed loop of few states, whose wave holds the control table, at the
table sizes where that form begins, wraps and ends (coast is the entry after
the last angle): every step's control is the one that the feedback call finds
at the step's state, and every step's state the oracle's FP64 plant step under
that control."""
import numpy as np
import pytest
import torch

from oracle.core import Oracle
from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu

STEPS, STATES = 5, 67


@pytest.mark.parametrize("model,drag", [("crown", 0.0), ("crown_euler", 0.0), ("orbit", 2e-3), ("eikonal", 0.0)])
@pytest.mark.parametrize("angles", [1, 2, 63, 64, 65, 127, 128])
def test_closed_loop_of_a_small_table(model, drag, angles):
    from paper_2407_14675_amd import dpo

    p = {
        "crown": lambda: inputs.crown_problem((12, 7, 9, 8), n_angles=angles),
        "crown_euler": lambda: inputs.crown_problem((12, 7, 9, 8), integrator="euler", n_angles=angles),
        "orbit": lambda: inputs.orbit_problem((9, 8, 7, 5), search=dict(mode="table", n_angles=angles)),
        "eikonal": lambda: inputs.eikonal_problem(9, n_angles=angles),
    }[model]()
    print("wave table", model, angles, flush=True)
    ctx, o = dpo.Context(p), Oracle(p)
    V = torch.from_numpy(inputs.random_value(p, seed=17, high=30.0, frac_M=0.0)).float().cuda()
    x0 = inputs.random_states(p, STATES, 19, margin=0.2)
    final, traj, thr, ang = ctx.simulate(V, x0, steps=STEPS, drag=drag)
    torch.cuda.synchronize()
    tau = p["dt"]
    differ = 0
    for s in range(STEPS):
        fa, ft = ctx.feedback(V, traj[s])[:2]
        torch.cuda.synchronize()
        differ += int(((fa != ang[s]) | (ft != thr[s])).sum())
        x, nxt = traj[s].cpu().numpy(), traj[s + 1].cpu().numpy()
        t, u = thr[s].cpu().numpy(), ang[s].cpu().numpy().astype(np.float64)
        for c in range(STATES):
            want = o.rk4_step(x[c], int(t[c]), u[c], tau, drag=drag)
            # about a hundred FP64 operations
            np.testing.assert_allclose(nxt[c], want, rtol=1e-12, atol=1e-12)
    # a tie in the last bit of a float32 Q may part the two searches
    assert differ <= 0.005 * STEPS * STATES
    assert torch.equal(final, traj[-1])
