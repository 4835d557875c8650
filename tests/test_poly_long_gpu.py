"""Long polynomials on 16 and 32 powers per column (s = 16 and 32): coefficients
beyond the small stage and beyond the large one, and few points, against Horner's
rule in binary64.  The powers carry 2^-17 each (two bfloat16 words), rounded
independently, so the error's norm over all points stays below 2^-17 of the
result's."""
import pytest
import torch

from paper_1908_06649_amd import inputs, tcu

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [16, 32])
@pytest.mark.parametrize("din,n,p", [("bf16", 1025, 3000), ("bf16", 17000, 262181),
                                     ("f16", 9000, 262144), ("bf16", 70000, 262149),
                                     ("f16", 3000, 70001)])
def test_poly_long(din, n, p, s):
    g = torch.Generator(device=gu.DEV).manual_seed(n + p)
    dt = inputs.TORCH_DTYPE[din]
    coef = torch.randn(n, generator=g, device=gu.DEV).to(dt)
    x = (torch.rand(p, generator=g, device=gu.DEV) * 2 - 1).to(dt)
    buf, out = gu.sentinel_buffer(p, torch.float32)
    tcu.tcu_poly_eval_ex(coef, n, x, p, out, s)
    torch.cuda.synchronize()
    assert gu.guard_intact(buf, p)
    xd = x.double()
    want = torch.zeros_like(xd)
    for a in reversed(coef.double().tolist()):
        want.mul_(xd).add_(a)
    assert ((out.double() - want).norm() / want.norm()).item() <= 2.0 ** -17
