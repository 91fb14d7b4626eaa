"""A solve whose curvature breaks down in a batch: a source that underflows in
the solver's storage gives <p, Ap> = 0, the call reports TM_ERR_NUMERIC, and
the batch's other solves keep the bits they have alone."""
import numpy as np
import pytest

from paper_1401_6749_amd import inputs
from tests import gpu_util as GU

pytestmark = pytest.mark.gpu


# 3 and 12 sources: one wave per neighbour direction, and the timeslice walk
# (64 reduction tiles a field)
@pytest.mark.parametrize("n", [3, 12])
@pytest.mark.parametrize("mode", ["mixed", "lp"])
def test_breakdown_leaves_the_other_slots_alone(mode, n):
    torch = GU.torch_mod()
    from paper_1401_6749_amd import tm

    dims = (8, 8, 8, 16)
    ctx, g = GU.context(), GU.load(dims, inputs.gauge_field(dims, seed=8))
    b = GU.to_dev(np.stack([inputs.random_spinor(dims, 90 + r) for r in range(n)]))
    b[1] *= 1e-60
    p = tm.solver_params(mode, tol=1e-8 if mode == "mixed" else 1e-2)
    x = torch.zeros_like(b)
    rc, st = tm.tm_cg_solve(ctx, g, 0.12, 0.01, p, n, b, x, check=False)
    assert rc == tm.TM_ERR_NUMERIC
    assert st[1]["iters"] == 0
    for r in (0, 2, n - 1):
        one = torch.zeros_like(b[:1])
        _, s1 = tm.tm_cg_solve(ctx, g, 0.12, 0.01, p, 1, b[r:r + 1].contiguous(), one)
        assert st[r]["iters"] == s1[0]["iters"] > 0
        assert torch.equal(x[r], one[0]), r
