"""The factorised sweep's two forms of a node (thrust feet in one cell, or in
several) and the order of its node list, through the C ABI: a sweep of the
whole grid, whose waves mostly take the one-cell form, against sweeps of
reduced grids of 60 random nodes, a single wave of both kinds of node that
takes the general form.  Values, angles and throttles are the same bit for
bit.  Sizes: below a wave's multiple, just above a chunk of the list (4096),
ten chunks with a ragged end; value fields that are smooth, rough with
patches of M, and a plateau with the target in it (the first sweep of a
solve)."""
import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu


def field(p, kind, target):
    if kind == "rough":
        V = inputs.random_value(p, seed=61, high=40.0, frac_M=0.1)
    elif kind == "plateau":
        V = np.full(target.shape, p["M"])
    else:
        ax = [np.linspace(p["lo"][k], p["hi"][k], p["n"][k]) for k in range(4)]
        R, VR, VT, MM = np.meshgrid(*ax, indexing="ij")
        V = (400 * (R - 1.05) ** 2 + 900 * VR ** 2 + 2000 * (VT - 0.976) ** 2 + 50 * (1 - MM)).transpose(3, 2, 1, 0)
    V = np.ascontiguousarray(V, dtype=np.float32)
    V[target] = 0.0
    return torch.from_numpy(V).cuda()


def sweep(ctx, V):
    W = V.clone()
    ang, thr = ctx.empty_policy()
    ctx.bellman_sweep(V, W, ang, thr)
    torch.cuda.synchronize()
    return W.cpu().numpy(), ang.cpu().numpy(), thr.cpu().numpy()


@pytest.mark.parametrize("search", ["table16", "table72", "scan_golden"])
@pytest.mark.parametrize("n", [(5, 3, 4, 2), (17, 8, 8, 4), (33, 11, 9, 13)])
def test_forms_agree_bit_for_bit(n, search):
    from paper_2407_14675_amd import dpo

    s = inputs.SCAN_GOLDEN if search == "scan_golden" else dict(mode="table", n_angles=int(search[5:]))
    p = inputs.orbit_problem(n, accel=1.7e-3, search=s)
    print("one-cell forms", n, search, flush=True)
    ctx = dpo.Context(p)
    kind = ctx.kind().cpu().numpy()
    rng = np.random.default_rng(62)
    for which in ("smooth", "rough", "plateau"):
        V = field(p, which, kind == 1)
        full = sweep(ctx, V)
        for _ in range(6):
            mask = np.zeros(kind.size, np.uint8)
            mask[rng.choice(kind.size, size=60, replace=False)] = 1
            some = mask.reshape(kind.shape) * (kind == 0) == 1
            one = dpo.Context(p, mask=torch.from_numpy(mask))
            for a, b in zip(full, sweep(one, V)):
                np.testing.assert_array_equal(a[some], b[some])
