"""The angle table of the one-cell waves of the scan + golden and seeded sweeps
(64 entries to a run, 128 to a stretch of LDS, 512 at most there, memory beyond) at the
table sizes where its place changes, through the C ABI: a sweep of the whole grid,
whose waves mostly take the one-cell form, against sweeps of reduced grids
of 60 random nodes, single waves of both kinds of node that take the general form and
have no such table.  Values, angles, throttles and the count of fallbacks are the same;
the grids' last waves are short.  A second, coarser scan after a fine one must not meet
the fine one's entries."""
import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu


def groups(free, rng, most):
    order = rng.permutation(np.flatnonzero(free))
    return [order[k:k + 60] for k in range(0, order.size, 60)][:most]


@pytest.mark.parametrize("mode", ["scan_golden", "seeded"])
@pytest.mark.parametrize("n", [(5, 3, 4, 2), (9, 6, 5, 4), (17, 8, 8, 8)])
def test_table_places(n, mode):
    from paper_2407_14675_amd import dpo

    p = inputs.orbit_problem(n, accel=1.7e-3, search=dict(mode="scan_golden", n_scan=64, n_golden=12))
    ctx = dpo.Context(p)
    kind = ctx.kind().cpu().numpy()
    free = kind.ravel() == 0
    rng = np.random.default_rng(64)
    few = groups(free, rng, 12)
    whole = sum(g.size for g in few) == free.sum()
    parts = []
    for g in few:
        mask = np.zeros(free.size, np.uint8)
        mask[g] = 1
        parts.append((dpo.Context(p, mask=torch.from_numpy(mask)), mask.reshape(kind.shape) == 1))
    ax = [np.linspace(p["lo"][k], p["hi"][k], n[k]) for k in range(4)]
    R, VR, VT, MM = np.meshgrid(*ax, indexing="ij")
    smooth = (400 * (R - 1.05) ** 2 + 900 * VR ** 2 + 2000 * (VT - 0.976) ** 2 + 50 * (1 - MM)).transpose(3, 2, 1, 0)
    rough = inputs.random_value(p, seed=65, high=40.0, frac_M=0.1)
    for n_scan in (8, 1024, 64, 65, 128, 129, 512, 513, 16):
        print("angles", n, mode, n_scan, flush=True)
        search = dict(inputs.SEEDED, n_scan=n_scan) if mode == "seeded" else dict(mode=mode, n_scan=n_scan, n_golden=12)
        for field in (smooth, rough):
            V = np.ascontiguousarray(field, np.float32)
            V[kind == 1] = 0.0
            V = torch.from_numpy(V).cuda()
            full = dict(mode="scan_golden", n_scan=n_scan, n_golden=12)
            ctx.set_search(full)
            best = [V.clone(), *ctx.empty_policy()]
            ctx.bellman_sweep(V, *best)
            seed = best[1] + torch.from_numpy(rng.normal(0, 0.2, kind.shape).astype(np.float32)).cuda()
            if mode == "seeded":
                # half of the nodes start at their searched value, which the local search finds again or not
                half = torch.from_numpy(rng.random(kind.shape) < 0.5).cuda()
                step = (best[0] - V).abs() / best[0].abs().clamp(min=1.0)
                search["fallback_tol"] = float(step[half].median())

            def sweep(c):
                c.set_search(search)
                out = [V.clone(), *c.empty_policy()]
                r = torch.zeros(5, dtype=torch.float64, device="cuda")
                if mode == "seeded":
                    c.bellman_sweep_seeded(V, *out, seed, resid=r)
                else:
                    c.bellman_sweep(V, *out, resid=r)
                torch.cuda.synchronize()
                return [t.cpu().numpy() for t in out], r.cpu().numpy()

            got, r = sweep(ctx)
            fallbacks = 0
            for c, some in parts:
                some = some & (kind == 0)
                part, rp = sweep(c)
                for a, b in zip(got, part):
                    np.testing.assert_array_equal(a[some], b[some])
                fallbacks += int(rp[4])
            if whole:
                assert fallbacks == int(r[4])
            if mode == "seeded":
                assert 0 < int(r[4]) < free.sum()
