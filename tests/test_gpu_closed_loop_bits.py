"""The closed loop's wave form (the control table held by the wave) and the
feedback call find the same control at every state of a trajectory, exactly: both
evaluate the same feet in the same operations and take the same first minimum."""
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["crown", "crown_euler", "orbit", "eikonal"])
def test_wave_table_and_feedback_agree_exactly(model):
    from paper_2407_14675_amd import dpo

    for angles in (1, 16, 63, 64, 72, 127):
        p = {
            "crown": lambda: inputs.crown_problem((12, 7, 9, 8), n_angles=angles),
            "crown_euler": lambda: inputs.crown_problem((12, 7, 9, 8), integrator="euler", n_angles=angles),
            "orbit": lambda: inputs.orbit_problem((9, 8, 7, 5), search=dict(mode="table", n_angles=angles)),
            "eikonal": lambda: inputs.eikonal_problem(9, n_angles=angles),
        }[model]()
        print("closed loop bits", model, angles, flush=True)
        ctx = dpo.Context(p)
        V = torch.from_numpy(inputs.random_value(p, seed=17, high=30.0)).float().cuda()
        x0 = inputs.random_states(p, 1000, 19, margin=0.05)
        _, traj, thr, ang = ctx.simulate(V, x0, steps=6, drag=2e-3 if model == "orbit" else 0.0)
        for s in range(6):
            fa, ft = ctx.feedback(V, traj[s])[:2]
            torch.cuda.synchronize()
            assert torch.equal(fa, ang[s]) and torch.equal(ft, thr[s])
