"""Timeslice walk on chunk shapes at the edges of its rule: partly filled
waves, chunks that span y or z, rows longer than a wave, extents of two, walks
of one timeslice and of several."""
import numpy as np
import pytest

from paper_1401_6749_amd import inputs
from tests import gpu_util as GU

pytestmark = pytest.mark.gpu

# (dims, right-hand sides): 240 of 256 lanes busy; 6 x 10 x 4 with a z halo;
# 36 sites of 64 lanes, T = 2; rows of 130 sites, one per chunk; many
# right-hand sides on a short lattice (a longer walk)
SHAPES = [((12, 10, 4, 6), 3), ((6, 10, 8, 2), 1), ((2, 6, 6, 4), 2), ((260, 4, 2, 2), 1), ((16, 4, 8, 6), 16)]
TOL = {"f64": 1e-14, "f32": 2e-6, "f16": 3e-3, "bf16": 2e-2}


@pytest.mark.parametrize("dims,nrhs", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_walk_shapes_match_oracle(oracle, dims, nrhs, prec):
    U = inputs.gauge_field(dims, seed=3)
    g = GU.load(dims, U)
    psi = np.stack([inputs.random_spinor(dims, 20 + r) for r in range(nrhs)])
    for op, dag in (("m", False), ("mdag", True)):
        got = GU.apply_op(g, op, 0.14, 0.02, prec, psi, dims)
        for r in (0, nrhs - 1):
            want = oracle.apply_M(dims, -1, U, 0.14, 0.02, psi[r], dag=dag)
            assert GU.relerr(got[r], want) < TOL[prec], (op, r)


@pytest.mark.parametrize("dims", [(12, 10, 4, 6), (2, 6, 6, 4)])
def test_walk_reductions_match_oracle(oracle, dims):
    """The CG sums over partly filled waves: same iteration count and iterate."""
    torch = GU.torch_mod()
    from paper_1401_6749_amd import tm

    U = inputs.gauge_field(dims, seed=4)
    g = GU.load(dims, U)
    eta = oracle.z4_source(dims, 8, 1)
    want, it, _, _ = oracle.solve(dims, -1, U, 0.12, 0.01, eta, tol=1e-10)
    b = GU.to_dev(eta[None])
    x = torch.zeros_like(b)
    _, st = tm.tm_cg_solve(GU.context(), g, 0.12, 0.01, tm.solver_params("f64", tol=1e-10), 1, b, x)
    assert st[0]["iters"] == it and st[0]["true_rel_resid"] < 1e-9
    assert GU.relerr(GU.from_dev(x[0]).reshape(want.shape), want) < 1e-11


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (12, 10, 4, 6)])
def test_split_equals_walk(prec, dims):
    """One right-hand side (one wave per neighbour direction) and sixteen of
    them (the walk: more tiles than one block per CU) give the same bits."""
    U = inputs.gauge_field(dims, seed=5)
    g = GU.load(dims, U)
    psi = np.stack([inputs.random_spinor(dims, 40 + r) for r in range(16)])
    for op in ("hop", "mhat_dag_mhat"):
        many = GU.apply_op(g, op, 0.14, 0.02, prec, psi, dims)
        for r in (0, 9):
            assert np.array_equal(many[r], GU.apply_op(g, op, 0.14, 0.02, prec, psi[r:r + 1], dims)[0]), (op, r)


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_full_operators_on_both_kernels(oracle, prec):
    """B H over both parities in one launch: split kernel (1), walk with the
    parities side by side (5) and one after the other (8 right-hand sides)."""
    dims = (8, 8, 6, 12)
    U = inputs.gauge_field(dims, seed=6)
    g = GU.load(dims, U)
    psi = np.stack([inputs.random_spinor(dims, 60 + r) for r in range(8)])
    want = oracle.apply_bh(dims, -1, U, 0.14, 0.02, psi[0])
    one = GU.apply_op(g, "bh", 0.14, 0.02, prec, psi[:1], dims)[0]
    assert GU.relerr(one, want) < TOL[prec]
    for n in (5, 8):
        got = GU.apply_op(g, "bh", 0.14, 0.02, prec, psi[:n], dims)
        assert np.array_equal(got[0], one)
        assert np.array_equal(got[n - 1], GU.apply_op(g, "bh", 0.14, 0.02, prec, psi[n - 1:n], dims)[0])
