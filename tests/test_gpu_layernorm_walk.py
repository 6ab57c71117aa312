"""LayerNorm over more rows than one pass of the chip takes (a half-wave then
walks several rows): the last partial pass, class-token rows met at any step of
the walk, and widths at and past the bound of the walking form."""
import numpy as np
import pytest

import oracle
from paper_2609_10018_amd import ffi, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import rel_err  # noqa: E402


@pytest.mark.parametrize("rows,d,tokens", [(10240, 64, 0), (10241, 64, 0), (20487, 200, 197),
                                           (30000, 768, 3), (10300, 256, 1), (11000, 1024, 197),
                                           (10999, 1032, 197)])
def test_layernorm_many_rows(rows, d, tokens):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator().manual_seed(rows + d)
    x = (torch.randn(rows, d, generator=g) * 2 + 0.5).bfloat16()
    gam, bet = 1 + 0.1 * torch.randn(d, generator=g), 0.1 * torch.randn(d, generator=g)
    xin, kw = x.double().numpy(), {}
    if tokens:
        cls = torch.randn((rows + tokens - 1) // tokens, d, generator=g)
        x[::tokens] = float("nan")  # class rows come from their own buffer alone
        xin[::tokens] = cls.double().numpy()
        kw = {"x_cls": cls.cuda(), "tokens": tokens}
    out = torch.empty(rows, d, dtype=torch.bfloat16, device="cuda")
    ffi.op_layernorm(inputs.BF16, x.cuda(), d, out, rows, d, gam.cuda(), bet.cuda(), 1e-6, **kw)
    got = out.float().cpu().numpy()
    ref = oracle.layer_norm(xin, gam.double().numpy(), bet.double().numpy(), 1e-6)
    assert np.isfinite(got).all()
    # One rounding to bf16, half a unit of 8 significant bits: up to 2^-8 = 3.9e-3 of
    # the largest value; the fp32 statistics add up to 1e-5.
    assert rel_err(got, ref) < 4e-3
