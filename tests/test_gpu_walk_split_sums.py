"""Split kernel and timeslice walk on the same work.  A launch of at most 512
reduction tiles x right-hand sides x parities takes the split kernel, a larger
one the walk; sizes here lie on both sides (tiles of a half field in brackets)."""
import numpy as np
import pytest

from paper_1401_6749_amd import inputs
from tests import gpu_util as GU

pytestmark = pytest.mark.gpu

# whole waves [64]; 240 of 256 lanes [96]; 120 of 128 lanes [252]; 36 of 64 lanes [96]
SOLVES = [((8, 8, 8, 16), 12), ((12, 10, 4, 24), 6), ((12, 10, 14, 18), 3), ((2, 6, 6, 96), 6)]


@pytest.mark.parametrize("mode", ["f64", "mixed", "lp"])
@pytest.mark.parametrize("dims,n", SOLVES)
def test_solves_alone_and_batched(oracle, dims, n, mode):
    """One source on the split kernel, n of them on the walk: the sums of the CG
    and of the true residual, the update of r, the same bits; and the oracle's
    iterate."""
    torch = GU.torch_mod()
    from paper_1401_6749_amd import tm

    U = inputs.gauge_field(dims, seed=11)
    ctx, g = GU.context(), GU.load(dims, U)
    eta = np.stack([oracle.z4_source(dims, 6, r) for r in range(n)])
    b = GU.to_dev(eta)
    p = tm.solver_params(mode, tol=1e-2, fixed_iters=5) if mode == "lp" else tm.solver_params(mode, tol=1e-10)
    x = torch.zeros_like(b)
    _, st = tm.tm_cg_solve(ctx, g, 0.12, 0.01, p, n, b, x)
    for r in (0, n - 1):
        one = torch.zeros_like(b[:1])
        _, s1 = tm.tm_cg_solve(ctx, g, 0.12, 0.01, p, 1, b[r:r + 1].contiguous(), one)
        assert st[r] == dict(s1[0], seconds=st[r]["seconds"]), r
        assert torch.equal(x[r], one[0]), r
    want, it, _, _ = oracle.solve(dims, -1, U, 0.12, 0.01, eta[0], **({"fixed_iters": 5} if mode == "lp" else {"tol": 1e-10}))
    if mode != "mixed":
        assert st[0]["iters"] == it
    if mode != "lp":
        assert st[0]["true_rel_resid"] < 1e-8
    assert GU.relerr(GU.from_dev(x[0]).reshape(want.shape), want) < {"f64": 1e-11, "mixed": 1e-8, "lp": 5e-3}[mode]


@pytest.mark.parametrize("half", ["f16", "bf16"])
@pytest.mark.parametrize("dims,n", [((8, 8, 8, 16), 12), ((12, 10, 14, 18), 3)])
def test_noise_solves_alone_and_batched(dims, n, half):
    """Noise solves whose right-hand side the last preparation Dslash writes
    (its norm and its half-precision stores), one and n to a launch."""
    from paper_1401_6749_amd import tm

    ctx, g = GU.context(), GU.load(dims, inputs.gauge_field(dims, seed=12))
    raw = []
    for batch in (1, n):
        p = tm.tsm_params(0.12, 0.01, 31, 0, n, lp=tm.solver_params("lp", fixed_iters=5, half=half), batch=batch)
        raw.append(tm.tm_loops_tsm(ctx, g, p, dims[3], want_raw=True)["raw_lp"])
    assert np.array_equal(raw[0], raw[1])


# right-hand sides of a half-field operator on the walk, then of a full one on
# the walk with the parities side by side (up to 6) and one after the other
OPERATORS = [((8, 8, 8, 16), 12, (5, 8)), ((12, 10, 14, 18), 3, (3, 8)), ((2, 6, 6, 96), 6, (6, 8))]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dims,half,full", OPERATORS)
def test_operators_alone_and_batched(dims, half, full, prec):
    g = GU.load(dims, inputs.gauge_field(dims, seed=13))
    psi = np.stack([inputs.random_spinor(dims, 50 + r) for r in range(max(half, *full))])
    for op, counts in (("mhat_dag_mhat", (half,)), ("m", full), ("bh", full)):
        for n in counts:
            many = GU.apply_op(g, op, 0.14, 0.02, prec, psi[:n], dims)
            for r in (0, n - 1):
                assert np.array_equal(many[r], GU.apply_op(g, op, 0.14, 0.02, prec, psi[r:r + 1], dims)[0]), (op, n, r)
