"""Kernels chosen on the smaller grids, at the edges of the rules that choose them."""
import numpy as np
import pytest
import torch

import fields
from oracle import multigrid as omg
from oracle.operator import face_coeffs_from_rho, project
from tests.gpu_helpers import dev, host, maxrel, raw_problem

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


@pytest.mark.parametrize("N", [32, 64])
@pytest.mark.parametrize("form", ["rho", "faces"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
def test_block_sweeps_against_oracle(N, form, dtype):
    """The finest grid swept in blocks, from the density (FP32 and FP64 at 64^3) and from
    face arrays (32^3, and any size set up from faces): sweeps of both orders and a cycle
    (restriction and prolongation inside the sweeps) against the oracle.  FP64 within
    1e-13 of the largest value for a sweep and 1e-12 for a cycle; FP32 within 2e-5 and
    1e-4, as the other FP32 kernels."""
    from paper_1410_2240_amd import MG, coeffs_from_rho
    inp = fields.make("c5", N)
    H = omg.setup(*face_coeffs_from_rho(inp.rho, inp.mask), inp.mask, inp.h)
    rho, mask = dev(inp.rho), dev(inp.mask)
    if form == "rho":
        mg = MG.from_rho(rho, mask, mixed=True)
    else:
        mg = MG(*coeffs_from_rho(rho, mask), mask, mixed=True)
    fp32 = dtype == torch.float32
    # 64^3 and up from rho: the FP32 faces come from the FP32 density
    lv32 = (omg.fp32_levels_from_rho(H, inp.rho) if form == "rho" and N >= 64 else omg.fp32_levels(H)) if fp32 else None
    lev = lv32[0] if fp32 else H.levels[0]
    g = np.random.default_rng(N)
    cast = np.float32 if fp32 else np.float64
    p = np.where(lev.mask, g.standard_normal(lev.bx.shape), 0.0).astype(cast)
    f = project(g.standard_normal(lev.bx.shape), lev.mask).astype(cast)
    for order in (0, 1):
        for sweeps in (1, 2):
            print(f"block sweep {N}^3 {form} {dtype} order={order} sweeps={sweeps}", flush=True)
            want = omg.smooth(p, f, lev, sweeps, (omg.RED, omg.BLACK) if order == 0 else (omg.BLACK, omg.RED))
            got = host(mg.smooth(0, dev(p), dev(f), sweeps, order))
            assert maxrel(got, want) <= (2e-5 if fp32 else 1e-13)
    want = omg.vcycle(H, p, f, lv32) if fp32 else omg.vcycle(H, p, f)
    assert maxrel(host(mg.vcycle(dev(p), dev(f))), want) <= (1e-4 if fp32 else 1e-12)


@pytest.mark.parametrize("N", [8, 16, 64])
def test_guess_and_means_with_a_body(N):
    """The passes over mask and vector around a solve, four cells to a thread: a guess that
    is NaN in the body is a guess of 0 there, the removed mean is the fluid mean of f, and
    the solution has none.  Both means to 1e-13 of the mean magnitude."""
    from paper_1410_2240_amd import MG
    g = np.random.default_rng(N)
    inp = fields.make("c2", N)
    mask = inp.mask.copy()
    mask[N // 4, 1:3, 1:4] = 0   # runs of 3: no group of four cells all alike
    live = mask != 0
    f = np.where(live, g.standard_normal(mask.shape) + 0.5, np.nan)
    p0 = np.where(live, g.standard_normal(mask.shape), np.nan)
    rho, m = dev(inp.rho), dev(mask)
    print(f"guess and means {N}^3", flush=True)
    mg = MG.from_rho(rho, m)
    p, hist, stats = mg.solve(dev(np.where(live, f, 0.0)), dev(p0), tol=1e-8)
    q, hist0, _ = mg.solve(dev(np.where(live, f, 0.0)), dev(np.where(live, p0, 0.0)), tol=1e-8)
    assert hist == hist0 and torch.equal(p, q)
    assert stats["active_cells"] == int(live.sum())
    assert abs(stats["removed_mean"] - f[live].mean()) <= 1e-13 * np.abs(f[live]).mean()
    out = host(p)
    assert (out[~live] == 0).all()
    assert abs(out[live].mean()) <= 1e-13 * np.abs(out[live]).mean()


@pytest.mark.parametrize("N", [8, 16])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("field", ["faces", "walls"])
def test_single_workgroup_cycle(N, dtype, field):
    """The cycle of one workgroup, from both of its top grids, against the oracle: from
    random face coefficients of contrast 1000 with a body (inactive cells on every grid),
    and with whole planes of closed cells at both walls.  Inactive cells keep what they
    held.  FP64 within 1e-12 of the largest value, FP32 within 1e-4."""
    from paper_1410_2240_amd import MG
    bx, by, bz, mask = raw_problem(N, 40 + N)
    if field == "walls":
        mask[0] = mask[-1] = 0
    H = omg.setup(bx, by, bz, mask, 1.0 / N)
    fp32 = dtype == torch.float32
    mg = MG(dev(bx), dev(by), dev(bz), dev(mask), mixed=True)
    g = np.random.default_rng(N)
    lev = H.levels[0]
    cast = np.float32 if fp32 else np.float64
    p = np.where(lev.mask, g.standard_normal(bx.shape), 0.0).astype(cast)
    f = project(g.standard_normal(bx.shape), lev.mask).astype(cast)
    print(f"single-workgroup cycle {N}^3 {dtype} {field}", flush=True)
    want = omg.vcycle(H, p, f, omg.fp32_levels(H)) if fp32 else omg.vcycle(H, p, f)
    got = host(mg.vcycle(dev(p), dev(f)))
    assert maxrel(got, want) <= (1e-4 if fp32 else 1e-12)
    kept = np.where(lev.mask, p, cast(7.0))
    got = host(mg.vcycle(dev(kept), dev(f)))
    assert (got[~lev.mask.astype(bool)] == 7.0).all()
    assert maxrel(np.where(lev.mask, got, 0), want) <= (1e-4 if fp32 else 1e-12)


@pytest.mark.parametrize("N", [8, 16, 32])
@pytest.mark.parametrize("case", ["open", "regions", "contrast"])
def test_setup_below_16_and_pseudo_inverse(N, case):
    """The setup's last launch, from each of its top grids: every grid's coefficients and
    mask against the oracle's, and the 4^3 solve against numpy's pseudo-inverse of the 4^3
    operator: without a body, with the fluid in two regions (a solid plane) and with face
    products over six decades.  The pseudo-inverse's error is its condition number (at most
    about 4e8 here) times eps: 1e-6 of the largest value; the faces within 1e-13."""
    from paper_1410_2240_amd import MG
    contrast = 1e6 if case == "contrast" else 1000.0
    bx, by, bz, mask = raw_problem(N, 70 + N, body=False, contrast=contrast)
    if case == "regions":
        mask[N // 2: N // 2 + N // 4] = 0   # a solid quarter: whole planes of the 4^3 grid
    H = omg.setup(bx, by, bz, mask, 1.0 / N)
    mg = MG(dev(bx), dev(by), dev(bz), dev(mask), mixed=True)
    print(f"setup {N}^3 {case}", flush=True)
    for l, lev in enumerate(H.levels):
        gx, gy, gz, gm = (host(t) for t in mg.level_coeffs(l))
        assert (gm.astype(bool) == lev.mask).all(), l
        for got, want in ((gx, lev.bx), (gy, lev.by), (gz, lev.bz)):
            assert maxrel(got, want) <= 1e-13, l
    lev = H.levels[-1]
    A = np.zeros((64, 64))
    for c in range(64):
        e = np.zeros(64)
        e[c] = 1.0
        A[:, c] = -omg.residual(e.reshape(4, 4, 4), np.zeros((4, 4, 4)), lev).ravel()
    live = lev.mask.ravel()
    f = np.where(live, np.random.default_rng(N).standard_normal(64), 0.0)
    g = np.where(live, f - f[live].mean(), 0.0)
    want = np.linalg.pinv(A, rcond=1e-13) @ g
    got = host(mg.coarse_solve(dev(f.reshape(4, 4, 4)))).ravel()
    assert np.abs(got - want).max() <= 1e-6 * np.abs(want).max()


def test_more_contexts_than_read_back_slots():
    """Seventy contexts at once (the pinned block has 64 slots): each solves, in any order
    of destruction, and slots are used again."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c2", 8)
    rho, mask, f = dev(inp.rho), dev(inp.mask), dev(inp.f)
    print("70 contexts", flush=True)
    want, hist, _ = MG.from_rho(rho, mask).solve(f, tol=1e-8)
    held = [MG.from_rho(rho, mask) for _ in range(70)]
    for order in (held[::3], held[1::3]):
        for mg in order:
            p, h, _ = mg.solve(f, tol=1e-8)
            assert h == hist and torch.equal(p, want)
    del held[::2]
    held += [MG.from_rho(rho, mask) for _ in range(20)]
    for mg in held:
        p, h, _ = mg.solve(f, tol=1e-8)
        assert h == hist and torch.equal(p, want)


@pytest.mark.parametrize("N", [8, 64])
@pytest.mark.parametrize("form", ["rho", "faces"])
def test_setup_pairs(N, form):
    """The finest grid's setup, two cells at a time: against the oracle on masks whose runs
    of one to three cells leave fluid cells with no open face, or with one on a high side
    only; with arrays that start 8 bytes (the mask one byte) past an aligned address; and a
    bad density or coefficient in either cell of a pair refused.  Faces within 1e-13."""
    from paper_1410_2240_amd import MG, MGError
    g = np.random.default_rng(90 + N)
    mask = (g.random((N, N, N)) < 0.35).astype(np.uint8)
    mask[:, : N // 2] |= (g.random((N, N // 2, N)) < 0.8).astype(np.uint8)
    mask[0, 0, :4] = mask[0, 1, :4] = mask[1, 0, :4] = 1
    rho = np.exp(g.uniform(np.log(1e-3), 0.0, (N, N, N)))
    bx, by, bz, _ = raw_problem(N, 91, body=False)
    if form == "rho":
        bx, by, bz = face_coeffs_from_rho(rho, mask)
    H = omg.setup(bx, by, bz, mask, 1.0 / N)

    def shifted(x):
        t = torch.empty(x.size + 1, dtype=torch.from_numpy(x).dtype, device="cuda")
        v = t[1:].view(x.shape)
        v.copy_(torch.from_numpy(x))
        return v

    print(f"setup pairs {N}^3 {form}", flush=True)
    m = shifted(mask)
    mg = MG.from_rho(shifted(rho), m) if form == "rho" else MG(shifted(bx), shifted(by), shifted(bz), m)
    for l, lev in enumerate(H.levels):
        gx, gy, gz, gm = (host(t) for t in mg.level_coeffs(l))
        assert (gm.astype(bool) == lev.mask).all(), l
        for got, want in ((gx, lev.bx), (gy, lev.by), (gz, lev.bz)):
            assert np.abs(got - want).max() <= 1e-13 * max(np.abs(want).max(), 1e-300), l
    live = np.argwhere(mask[2, 2] != 0)[:, 0]
    for i in (int(live[live % 2 == 0][0]), int(live[live % 2 == 1][0])):
        for value in (np.nan, -1.0):
            rho2, bx2 = rho.copy(), bx.copy()
            rho2[2, 2, i] = bx2[2, 2, i] = value
            full = np.ones_like(mask)
            with pytest.raises(MGError):
                if form == "rho":
                    MG.from_rho(dev(rho2), dev(full))
                else:
                    MG(dev(bx2), dev(by), dev(bz), dev(full))


@pytest.mark.parametrize("N", [128, 256])
def test_norm_passes_through_lds(N):
    """The residual norm and the mixed update + residual pass with their stencil through
    LDS (128^3, the smallest; 256^3, two tiles to a row): the first residual of a guess
    against the face-array context's, bit for bit (its pass reads neighbours from the
    caches), and a mixed refinement against FP64, within 1e-9."""
    from paper_1410_2240_amd import MG, coeffs_from_rho
    inp = fields.make("c2", N)
    rho, mask, f = dev(inp.rho), dev(inp.mask), dev(inp.f)
    g = torch.Generator(device="cuda").manual_seed(N)
    p0 = torch.randn(rho.shape, generator=g, device="cuda", dtype=torch.float64)
    print(f"norm passes {N}^3", flush=True)
    a = MG.from_rho(rho, mask)
    b = MG(*coeffs_from_rho(rho, mask), mask)
    _, ha, _ = a.solve(f, p0.clone(), max_cycles=0, raise_on_fail=False)
    _, hb, _ = b.solve(f, p0.clone(), max_cycles=0, raise_on_fail=False)
    assert ha == hb and len(ha) == 1
    m = MG.from_rho(rho, mask, mixed=True)
    pm, hm, _ = m.solve(f, p0.clone(), tol=1e-12, max_cycles=80)
    pa, _, _ = a.solve(f, p0.clone(), tol=1e-12, max_cycles=80)
    assert hm[0] == ha[0]
    assert float((pm - pa).norm() / pa.norm()) <= 1e-9


@pytest.mark.parametrize("N", [8, 16])
def test_small_solve_in_one_launch(N):
    """FP64 V-cycles on the grids solved in one launch: the history cycle by cycle against
    the oracle's (to 1e-6 of each entry, down to 1e-8 where rounding takes over), more
    entries than come back with the scalars, a warm start, and the ways to end: no
    convergence, no cycles allowed, f constant, f not finite, an item of a batch on a lane."""
    from paper_1410_2240_amd import MG, MGError
    inp = fields.make("c2", N)
    H = omg.setup(*face_coeffs_from_rho(inp.rho, inp.mask), inp.mask, inp.h)
    rho, mask, f = dev(inp.rho), dev(inp.mask), dev(inp.f)
    mg = MG.from_rho(rho, mask)
    print(f"small solve {N}^3", flush=True)
    p, hist, stats = mg.solve(f, tol=1e-30, max_cycles=150, raise_on_fail=False)
    assert stats["status"] == -4 and stats["cycles"] == 150 and len(hist) == 151
    _, want = omg.solve(H, inp.f, tol=1e-9, max_cycles=60)
    for got, ref in zip(hist, want):
        if ref > 1e-8:
            assert abs(got - ref) <= 1e-6 * ref
    assert max(hist[40:]) <= 1e-12
    q, again, stats = mg.solve(f, p.clone(), tol=1e-10)
    assert stats["cycles"] == 0 and len(again) == 1
    assert float((p - q).abs().max()) <= 1e-13 * float(p.abs().max())
    q, one, stats = mg.solve(f, tol=1e-10, max_cycles=0, raise_on_fail=False)
    assert stats["status"] == -4 and one == hist[:1] and float(q.abs().max()) == 0.0
    q, zero, stats = mg.solve(torch.full_like(f, 3.0), torch.ones_like(f))
    assert stats["status"] == 0 and zero == [0.0] and float(q.abs().max()) == 0.0
    bad = f.clone()
    bad[tuple(int(x) for x in np.argwhere(inp.mask != 0)[5])] = float("nan")
    with pytest.raises(MGError):
        mg.solve(bad)
    batch = torch.stack([f, 2.0 * f, torch.flip(f, [2]) * mask])
    pl, hl, _ = MG.from_rho(rho, mask, lanes=2).solve(batch, tol=1e-9)
    for b in range(3):
        pb, hb, _ = mg.solve(batch[b].contiguous(), tol=1e-9)
        assert hb == hl[b] and torch.equal(pb, pl[b])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("N", [128, 256])
def test_correction_inside_the_post_smoothing(N, dtype):
    """A cycle whose post-smoothing pass adds the coarse correction itself (256^3; at 128^3
    it has a pass of its own) against the same cycle step by step, bit for bit: two sweeps,
    restriction, a cycle of the hierarchy one grid down, prolongation, two sweeps.  The
    field has its body and both walls in reach of the interpolation."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c5", N)
    mg = MG.from_rho(dev(inp.rho), dev(inp.mask), mixed=True)
    p, f = random_pair(inp, N, dtype)
    print(f"correction inside post-smoothing {N}^3 {dtype}", flush=True)
    got = mg.vcycle(p.clone(), f)
    bx, by, bz, mask = mg.level_coeffs(1)
    below = MG(bx, by, bz, mask, h=2.0 / N, mixed=True)
    want = mg.smooth(0, p.clone(), f, 2, 0)
    fc = mg.residual_restrict(0, want, f)
    ec = below.vcycle(torch.zeros_like(fc), fc)
    want = mg.smooth(0, mg.prolong_add(0, ec, want), f, 2, 1)
    assert torch.equal(got, want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("N", [128, 256])
def test_two_sweep_pass_from_face_arrays(N, dtype):
    """The two-sweep pass reading face arrays (FP32 from 256^3) against one-pass sweeps, bit
    for bit: random faces of contrast 1000 with a body, the bottom wall and the top one, both
    orders, even and odd counts."""
    from paper_1410_2240_amd import MG
    bx, by, bz, mask = raw_problem(N, N)
    mg = MG(dev(bx), dev(by), dev(bz), dev(mask), mixed=True)
    g = torch.Generator(device="cuda").manual_seed(N)
    live = mg.level_coeffs(0)[3].bool()
    for order in (0, 1):
        for sweeps in (2, 3, 4):
            print(f"two-sweep pass, faces {N}^3 {dtype} order={order} sweeps={sweeps}", flush=True)
            p, f = (torch.randn(bx.shape, generator=g, device="cuda", dtype=dtype) * live for _ in range(2))
            got = mg.smooth(0, p.clone(), f, sweeps, order)
            want = p.clone()
            for _ in range(sweeps):
                want = mg.smooth(0, want, f, 1, order)
            assert torch.equal(got, want), (order, sweeps)


@pytest.mark.parametrize("N", [32, 64])
@pytest.mark.parametrize("form", ["rho", "faces"])
def test_direction_pass_one_pair_per_thread(N, form):
    """The flexible-CG direction pass of 32^3 and 64^3, from both forms of the coefficients:
    FP64 histories step by step against the oracle's (to 1e-5 of each entry: rounding of
    1e-16 times the residual's fall to 1e-7 and its growth over the recurrences), a warm
    start, and mixed preconditioning (FP32 z) to the same solution."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c2", N)
    faces = face_coeffs_from_rho(inp.rho, inp.mask)
    H = omg.setup(*faces, inp.mask, inp.h)
    f = dev(inp.f)
    make = lambda **kw: (MG.from_rho(dev(inp.rho), dev(inp.mask), krylov=True, **kw) if form == "rho"
                         else MG(*(dev(b) for b in faces), dev(inp.mask), krylov=True, **kw))
    print(f"direction pass {N}^3 {form}", flush=True)
    p, hist, _ = make().solve(f, tol=1e-11, max_cycles=60)
    want_p, want = omg.solve_fcg(H, inp.f, tol=1e-11, max_iters=60)[:2]
    for got, ref in zip(hist, want):
        if ref > 1e-7:
            assert abs(got - ref) <= 1e-5 * ref
    assert maxrel(host(p), want_p) <= 1e-8
    q, again, _ = make().solve(f, 0.5 * p, tol=1e-11, max_cycles=60)
    assert abs(again[0] - 0.5) <= 1e-9 and maxrel(host(q), want_p) <= 1e-8
    q, mixed, _ = make(mixed=True).solve(f, tol=1e-11, max_cycles=60)
    assert maxrel(host(q), want_p) <= 1e-8 and abs(len(mixed) - len(hist)) <= 2


@pytest.mark.parametrize("N", [32, 64])
@pytest.mark.parametrize("form", ["rho", "faces"])
def test_norm_pass_one_pair_per_thread(N, form):
    """The residual norm of 32^3 and 64^3, from both forms of the coefficients: V-cycle
    histories against the oracle's (to 1e-6 of each entry down to 1e-8, where rounding takes
    over), a source with a mean, a warm start, and the FP32 copy that a mixed solve takes."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c2", N)
    faces = face_coeffs_from_rho(inp.rho, inp.mask)
    H = omg.setup(*faces, inp.mask, inp.h)
    src = inp.f + 0.25 * np.abs(inp.f).max()
    f = dev(src)
    make = lambda **kw: (MG.from_rho(dev(inp.rho), dev(inp.mask), **kw) if form == "rho"
                         else MG(*(dev(b) for b in faces), dev(inp.mask), **kw))
    print(f"norm pass {N}^3 {form}", flush=True)
    p, hist, _ = make().solve(f, tol=1e-11, max_cycles=100)
    want_p, want = omg.solve(H, src, tol=1e-11, max_cycles=100)
    for got, ref in zip(hist, want):
        if ref > 1e-8:
            assert abs(got - ref) <= 1e-6 * ref
    assert maxrel(host(p), want_p) <= 1e-8
    _, again, _ = make().solve(f, 0.5 * p, tol=1e-11, max_cycles=100)
    assert abs(again[0] - 0.5) <= 1e-9
    q, mixed, _ = make(mixed=True).solve(f, tol=1e-11, max_cycles=100)
    assert maxrel(host(q), want_p) <= 1e-8 and abs(len(mixed) - len(hist)) <= 2
