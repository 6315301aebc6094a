"""Power of the FP32 transform of white noise against FP64: the rounding of the butterflies' constants takes a
part of it, the same for every mode, that no average over modes removes."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,most", [(128, 1.45e-7), (256, 1.25e-7), (512, 1.45e-7)])
def test_fp32_transform_keeps_its_power(gpu, n, most):
    """Most: what constants and twiddles rounded to 24 bits lack with radices of 8 and below, from their norms: a
    column axis 4.07e-8, 4.12e-8, 4.84e-8, the half-length z axis 3.77e-8, 4.07e-8, 4.12e-8 and its split up to
    half the twiddles' mean norm: 1.3, 1.2 and 1.35e-7 in all; radix 16 with rounded constants takes 1.45e-7 at
    256.  The noise of the roundings themselves averages to 1e-10."""
    import torch
    from paper_1704_02357_amd import Plan
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(n, n, n, generator=g, device="cuda", dtype=torch.float32)
    out = torch.empty(n, n, n // 2, 2, device="cuda", dtype=torch.float32)
    print(f"[case] fft power side {n}", flush=True)
    plan = Plan(n, 100.0, precision=0)
    plan.fft3d_forward(x, out)
    plan.close()
    ref = torch.fft.rfftn(x.double())[..., : n // 2]
    w = torch.full((n // 2,), 2.0, device="cuda", dtype=torch.float64)
    w[0] = 1.0
    p32 = ((out.double() ** 2).sum(-1) * w).sum().item()
    p64 = ((ref.real ** 2 + ref.imag ** 2) * w).sum().item()
    print(f"[fft power] side {n} {p32 / p64 - 1:.3e}", flush=True)
    assert abs(p32 / p64 - 1) <= most
