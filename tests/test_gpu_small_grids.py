"""Kernels chosen on the smaller grids, at the edges of the rules that choose them."""
import pytest
import torch

import fields
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu


def random_pair(inp, seed, dtype):
    g = torch.Generator(device="cuda").manual_seed(seed)
    live = dev(inp.mask).bool()
    return tuple(torch.randn(inp.rho.shape, generator=g, device="cuda", dtype=dtype) * live for _ in range(2))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
def test_two_sweep_pass_128(dtype):
    """The smallest grid of the two-sweep pass (8-plane chunks; in FP32 one tile spans a
    row, so its halo is the tile itself): two sweeps in one pass against two one-pass
    sweeps, bit for bit, both orders, an even and an odd count."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c5", 128)
    mg = MG.from_rho(dev(inp.rho), dev(inp.mask), mixed=True)
    for order in (0, 1):
        for sweeps in (2, 3):
            print(f"two-sweep pass 128^3 {dtype} order={order} sweeps={sweeps}", flush=True)
            p, f = random_pair(inp, 10 * sweeps + order, dtype)
            got = mg.smooth(0, p.clone(), f, sweeps, order)
            want = p.clone()
            for _ in range(sweeps):
                want = mg.smooth(0, want, f, 1, order)
            assert torch.equal(got, want)


@pytest.mark.parametrize("lanes", [1, 2, 5])
def test_two_sweep_pass_128_concurrent(lanes):
    """Right-hand sides solved at once sweep in longer z-chunks (16, 16 and 32 planes here):
    the same bits as one at a time."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c2", 128)
    f = dev(fields.batch_rhs(inp.mask, lanes + 1))
    rho, mask = dev(inp.rho), dev(inp.mask)
    print(f"two-sweep pass 128^3, {lanes} lanes", flush=True)
    p, hist, _ = MG.from_rho(rho, mask, lanes=lanes).solve(f, tol=1e-6, max_cycles=60, raise_on_fail=False)
    q, hist1, _ = MG.from_rho(rho, mask).solve(f, tol=1e-6, max_cycles=60, raise_on_fail=False)
    assert hist == hist1
    assert torch.equal(p, q)
