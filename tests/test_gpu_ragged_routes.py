"""Kernels that share the work of a ragged lattice: solves whose precisions run
on different kernels with different reduction tiles, and single half-precision
right-hand sides."""
import numpy as np
import pytest

from paper_1401_6749_amd import inputs
from tests import gpu_util as GU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["f64", "mixed", "lp"])
def test_solves_on_few_busy_lanes(oracle, mode):
    """34 x 34 x 2 x 8: the register kernel in FP64 and half precision, the walk
    with partly filled waves in FP32 (272 tiles, the register kernel's 145)."""
    torch = GU.torch_mod()
    from paper_1401_6749_amd import tm

    dims, n = (34, 34, 2, 8), 4
    U = inputs.gauge_field(dims, seed=9)
    ctx, g = GU.context(), GU.load(dims, U)
    eta = np.stack([oracle.z4_source(dims, 5, r) for r in range(n)])
    b = GU.to_dev(eta)
    p = tm.solver_params(mode, tol=1e-2, fixed_iters=5) if mode == "lp" else tm.solver_params(mode, tol=1e-10)
    x = torch.zeros_like(b)
    _, st = tm.tm_cg_solve(ctx, g, 0.12, 0.01, p, n, b, x)
    want, it, _, _ = oracle.solve(dims, -1, U, 0.12, 0.01, eta[1], **({"fixed_iters": 5} if mode == "lp" else {"tol": 1e-10}))
    assert GU.relerr(GU.from_dev(x[1]).reshape(want.shape), want) < {"f64": 1e-11, "mixed": 1e-8, "lp": 5e-3}[mode]
    if mode != "mixed":
        assert st[1]["iters"] == it
    for r in range(n):
        one = torch.zeros_like(b[:1])
        _, s1 = tm.tm_cg_solve(ctx, g, 0.12, 0.01, p, 1, b[r:r + 1].contiguous(), one)
        assert st[r] == dict(s1[0], seconds=st[r]["seconds"]), r
        assert torch.equal(x[r], one[0]), r


@pytest.mark.parametrize("prec", ["f16", "bf16"])
def test_one_half_precision_source(prec):
    """18^3 x 12 (576 tiles): one right-hand side on the register kernel, three on
    the walk, the same bits."""
    dims = (18, 18, 18, 12)
    g = GU.load(dims, inputs.gauge_field(dims, seed=10))
    psi = np.stack([inputs.random_spinor(dims, 30 + r) for r in range(3)])
    for op in ("mhat", "mhat_dag_mhat"):
        many = GU.apply_op(g, op, 0.14, 0.02, prec, psi, dims)
        for r in (0, 2):
            assert np.array_equal(many[r], GU.apply_op(g, op, 0.14, 0.02, prec, psi[r:r + 1], dims)[0]), (op, r)
