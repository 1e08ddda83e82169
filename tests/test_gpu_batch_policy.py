"""The batched solve's policy arrays: written at the free nodes, with the policy of the
problems solved one after another, and left as the caller made them at the fixed
ones, whatever device memory held before."""
import numpy as np
import pytest
import torch

from paper_2407_14675_amd import inputs

pytestmark = pytest.mark.gpu


def test_fixed_nodes_keep_the_callers_policy():
    from paper_2407_14675_amd import dpo

    print("batch policy", flush=True)
    probs = [inputs.with_grid(p, (side,) * 4) for p, side in zip(inputs.batch_problems(3), (9, 12, 7))]
    b = dpo.Batch(probs)
    V, W = b.init_values(), b.init_values()
    angs, thrs = b.empty_policies()
    a2, t2 = b.empty_policies()
    for a, t in zip(angs, thrs):
        a.fill_(7.5)
        t.fill_(9)
    b.solve_vi(V, angs, thrs, tol_rel=0.0, max_sweeps=16, sweeps_per_graph=8)
    b.solve_sequential(W, a2, t2, tol_rel=0.0, max_sweeps=16, check_every=16)
    torch.cuda.synchronize()
    for p, x in enumerate(probs):
        fixed = dpo.Context(x).kind().cpu().numpy() != 0
        assert fixed.any() and not fixed.all()
        np.testing.assert_array_equal(V[p].cpu().numpy(), W[p].cpu().numpy())
        for got, want, kept in ((angs[p], a2[p], 7.5), (thrs[p], t2[p], 9)):
            got, want = got.cpu().numpy(), want.cpu().numpy()
            np.testing.assert_array_equal(got[~fixed], want[~fixed])
            assert (got[fixed] == kept).all()
