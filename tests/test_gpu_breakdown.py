"""A residual that is not finite ends a solve as a breakdown, the first one too."""
import numpy as np
import pytest
import torch

import fields
from tests.gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed,krylov", [(False, False), (True, False), (False, True), (True, True)],
                         ids=["v", "mixed_v", "cg", "mixed_cg"])
@pytest.mark.parametrize("N", [8, 16, 64])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_guess_that_is_not_finite(N, mixed, krylov, value):
    """A NaN or an infinity in a fluid cell of the guess: MG_EBREAKDOWN with the first
    residual alone in the history and in the statistics, not a converged solve; the items
    around it in a batch, one at a time and on lanes, are what they are by themselves."""
    from paper_1410_2240_amd import MG, MGError
    from paper_1410_2240_amd._lib import MG_EBREAKDOWN
    inp = fields.make("c2", N)
    rho, mask = dev(inp.rho), dev(inp.mask)
    print(f"guess {value} {N}^3 mixed={mixed} krylov={krylov}", flush=True)
    mg = MG.from_rho(rho, mask, mixed=mixed, krylov=krylov)
    f = dev(inp.f)
    cell = tuple(int(x) for x in np.argwhere(inp.mask != 0)[7])
    bad = torch.zeros_like(f)
    bad[cell] = value
    with pytest.raises(MGError) as e:
        mg.solve(f, bad.clone(), tol=1e-8)
    assert e.value.code == MG_EBREAKDOWN
    _, hist, stats = mg.solve(f, bad.clone(), tol=1e-8, raise_on_fail=False)
    assert stats["status"] == MG_EBREAKDOWN and stats["cycles"] == 0
    assert len(hist) == 1 and not np.isfinite(hist[0])
    assert not np.isfinite(stats["final_relres"])
    want, hist0, _ = mg.solve(f, tol=1e-8)
    batch, guess = torch.stack([f, f, f]), torch.stack([torch.zeros_like(f), bad, torch.zeros_like(f)])
    for m in (mg, MG.from_rho(rho, mask, mixed=mixed, krylov=krylov, lanes=2)):
        p, hists, stats = m.solve(batch, guess.clone(), tol=1e-8, raise_on_fail=False)
        assert stats["status"] == MG_EBREAKDOWN and not np.isfinite(stats["final_relres"])
        assert hists[0] == hist0 and hists[2] == hist0 and len(hists[1]) == 1
        assert torch.equal(p[0], want) and torch.equal(p[2], want)
