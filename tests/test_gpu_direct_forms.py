"""The direct sweeps' two forms, cell cache and keyed corners, on grids above the sizes
from which the cell cache is taken: the sweep of the whole grid against sweeps of
reduced grids of the same problem, too small for it.  Values, angles and
throttles are the same bit for bit at every node of the reduced grids, which hold random
nodes, many of them on the domain's faces; odd sides put a row of nodes on v_r = 0,
whose feet hover about a face."""
import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu

TABLE = dict(mode="table", n_angles=40)
CASES = {
    "crown_heun": (inputs.crown_problem((64, 17, 18, 18), n_angles=40), TABLE),
    "orbit_heun": (dict(inputs.orbit_problem((31, 23, 22, 22)), integrator="heun"), TABLE),
    "orbit_euler": (inputs.orbit_problem((25, 21, 19, 18)), TABLE),
    "orbit_euler_scan": (inputs.orbit_problem((25, 21, 19, 18)), inputs.SCAN_GOLDEN),
    "orbit_euler_seeded": (inputs.orbit_problem((25, 21, 19, 18)), dict(inputs.SEEDED, fallback_tol=1e-2)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_forms_agree_bit_for_bit(case):
    from paper_2407_14675_amd import dpo

    p, search = CASES[case]
    p = dict(p, search=dict(search))
    print("direct forms", case, flush=True)
    ctx = dpo.Context(p)
    ctx.set_kernel_path(1)
    kind = ctx.kind().cpu().numpy()
    rng = np.random.default_rng(81)
    i = np.indices(kind.shape)
    face = sum(((i[k] == 0) | (i[k] == kind.shape[k] - 1)).astype(int) for k in range(4))
    seed = torch.from_numpy(rng.uniform(-np.pi, np.pi, kind.shape).astype(np.float32)).cuda()

    def sweep(c, V):
        c.set_kernel_path(1)
        out = [V.clone(), *c.empty_policy()]
        if search["mode"] == "seeded":
            c.bellman_sweep_seeded(V, *out, seed)
        else:
            c.bellman_sweep(V, *out)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    masks = [(rng.random(kind.shape) < 0.03 + 0.05 * face).astype(np.uint8) for _ in range(2)]
    parts = [(dpo.Context(p, mask=torch.from_numpy(m.ravel())), (m == 1) & (kind == 0)) for m in masks]
    for c, some in parts:
        assert 5000 < some.sum() < 100000
    smooth = 40.0 * sum(((i[k] - 0.4 * kind.shape[k]) / kind.shape[k]) ** 2 for k in range(4))
    for field in (smooth, inputs.random_value(p, seed=82, high=30.0, frac_M=0.05)):
        V = np.ascontiguousarray(field, np.float32)
        V[kind == 1] = 0.0
        V = torch.from_numpy(V).cuda()
        full = sweep(ctx, V)
        for c, some in parts:
            for a, b in zip(full, sweep(c, V)):
                np.testing.assert_array_equal(a[some], b[some])
