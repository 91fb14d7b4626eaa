"""Load policies of the direction update: 1, 6 and 16 FP16 fields of 17 MB take
ordinary loads, streamed x and r, and all loads streamed; every field has the
bits of the update on that field alone."""
import pytest

from paper_1401_6749_amd import inputs
from tests import gpu_util as GU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [6, 16])
def test_update_same_bits_for_every_load_policy(nrhs):
    torch = GU.torch_mod()
    from paper_1401_6749_amd import tm

    dims = (32, 32, 32, 20)
    ctx = GU.context()
    g = GU.load(dims, inputs.unit_gauge(dims), precs=("f16",))
    hb = tm.tm_field_bytes(g, "f16", full=False)
    gen = torch.Generator(device="cuda").manual_seed(3)

    def fields():
        out = torch.empty(nrhs, hb, dtype=torch.uint8, device="cuda")
        full = torch.empty(2 * hb, dtype=torch.uint8, device="cuda")
        for i in range(nrhs):
            c = torch.randn(2 * hb // 52, 4, 3, 2, dtype=torch.float64, device="cuda", generator=gen)
            tm.tm_field_import(ctx, g, "f16", 1, c, full)
            out[i] = full[:hb]
        return out

    p, r, x = fields(), fields(), fields()
    alpha, beta = [0.1 + 0.01 * i for i in range(nrhs)], [0.9 - 0.02 * i for i in range(nrhs)]
    p1, x1 = p.clone(), x.clone()
    tm.tm_cg_update(ctx, g, "f16", nrhs, p, r, x, hb, alpha, beta)
    for i in range(nrhs):
        tm.tm_cg_update(ctx, g, "f16", 1, p1[i], r[i], x1[i], hb, alpha[i:i + 1], beta[i:i + 1])
    torch.cuda.synchronize()
    assert torch.equal(p, p1) and torch.equal(x, x1)
    tm.tm_free_gauge(ctx, g)
