"""The coarse correction added inside the post-smoothing pass, near the end of the range of
its type."""
import math

import pytest
import torch

import fields
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("N", [128, 256])
def test_cycle_scales_by_powers_of_two(N, dtype):
    """A cycle is linear and scaling by a power of two is exact, so f times 2^k gives p times
    2^k bit for bit as long as nothing overflows or is subnormal.  With faces of 1/rho = 2^-10
    nothing but the correction comes near p's own size, and p is taken to within a factor of
    16 of the largest value of the type (256^3: the correction inside the post-smoothing;
    128^3: a pass of its own)."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c5", N)
    mask = dev(inp.mask)
    rho = torch.full((N, N, N), 1024.0, device="cuda", dtype=torch.float64)
    mg = MG.from_rho(rho, mask, h=1.0, mixed=True)
    x = (torch.arange(N, device="cuda", dtype=torch.float64) + 0.5) * (2 * math.pi / N)
    f = (torch.cos(x)[None, None, :] + torch.sin(x)[None, :, None] + torch.cos(x / 2)[:, None, None]) * (mask != 0)
    f = (f - f.sum() / (mask != 0).sum()) * (mask != 0)
    f = f.to(dtype)
    print(f"cycle scaled {N}^3 {dtype}", flush=True)
    want = mg.vcycle(torch.zeros_like(f), f)
    top = 127 if dtype == torch.float32 else 1023
    k = top - 3 - math.frexp(float(want.abs().max()))[1]
    half = k // 2   # 2^k itself may be out of range
    scale = lambda t: t * 2.0 ** half * 2.0 ** (k - half)
    got = mg.vcycle(torch.zeros_like(f), scale(f))
    assert torch.equal(got, scale(want))
