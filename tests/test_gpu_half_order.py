"""Half precision on lattices without a chunk of whole waves on aligned tiles:
the operators give the register kernel's bits on every kernel."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1401_6749_amd import inputs
from tests import gpu_util as GU

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# one right-hand side: one wave per neighbour direction on the small lattices;
# many: the timeslice walk, with whole waves (24^3) and partly filled ones
SHAPES = [((12, 10, 4, 6), (1, 16)), ((24, 24, 24, 4), (1, 2)), ((12, 10, 14, 18), (1, 5))]
OPS = ("hop", "mdag", "mhat", "mhat_dag_mhat")


def _apply(dims, prec, nrhs):
    g = GU.load(dims, inputs.gauge_field(dims, seed=7))
    psi = np.stack([inputs.random_spinor(dims, 80 + r) for r in range(nrhs)])
    return [GU.apply_op(g, op, 0.15, 0.02, prec, psi, dims) for op in OPS]


CHILD = r"""
import sys
import numpy as np
sys.path.insert(0, sys.argv[1])
from tests import test_gpu_half_order as T
out = {}
for dims, counts in T.SHAPES:
    for prec in ("f16", "bf16"):
        for k, v in enumerate(T._apply(dims, prec, max(counts))):
            out["%d_%s_%d" % (dims[3], prec, k)] = v
    print(dims, "done", flush=True)
np.savez(sys.argv[2], **out)
"""


@pytest.fixture(scope="module")
def register_kernel(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("half") / "reg.npz")
    p = subprocess.run([sys.executable, "-u", "-c", CHILD, ROOT, out], env=dict(os.environ, TM_LDS_WALK="0"),
                       capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-2000:]
    return np.load(out)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["f16", "bf16"])
@pytest.mark.parametrize("dims,counts", SHAPES)
def test_half_operators_keep_the_register_kernels_bits(register_kernel, dims, counts, prec):
    for n in counts:
        for k, got in enumerate(_apply(dims, prec, n)):
            want = register_kernel["%d_%s_%d" % (dims[3], prec, k)][:n]
            assert np.array_equal(got, want), (OPS[k], n, GU.relerr(got, want))
