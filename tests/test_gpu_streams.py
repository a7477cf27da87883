"""Contexts used on more than one stream."""
import pytest
import torch

import fields
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("N", [8, 16, 32, 128])
def test_a_setup_is_done_when_it_returns(N, mixed):
    """Set up on one stream and used at once on another, nothing between them: the coarsest
    solve (the pseudo-inverse), every grid's coefficients and a solve are those of a context
    used on the stream it was set up on."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c2", N)
    rho, mask, f = dev(inp.rho), dev(inp.mask), dev(inp.f)
    g = torch.Generator(device="cuda").manual_seed(N)
    fc = torch.randn((4, 4, 4), generator=g, device="cuda", dtype=torch.float64)
    side = torch.cuda.Stream()
    make = lambda: MG.from_rho(rho, mask, mixed=mixed)

    def used(mg):
        return [mg.coarse_solve(fc)] + [t for l in range(mg.levels) for t in mg.level_coeffs(l)] + \
               [mg.solve(f, tol=1e-9)[0]]

    want = used(make())
    torch.cuda.synchronize()
    for repeat in range(5):
        print(f"setup on another stream {N}^3 mixed={mixed} {repeat}", flush=True)
        with torch.cuda.stream(side):
            mg = make()
        got = used(mg)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
