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


def pending(stream):
    """Work of some 40 ms on the stream, and an event after it."""
    torch.cuda._sleep(100_000_000)
    return stream.record_event()


@pytest.mark.parametrize("lanes", [0, 2])
@pytest.mark.parametrize("N", [16, 128])
def test_workspace_is_kept_for_another_stream(N, lanes):
    """Built on one stream, solved and applied on another, dropped while that one has work
    to do, and memory of the workspace's size allocated and filled on the first at once: the
    results are those of a context used on one stream."""
    from paper_1410_2240_amd import MG
    inp = fields.make("c2", N)
    rho, mask, f = dev(inp.rho), dev(inp.mask), dev(fields.batch_rhs(inp.mask, 3))
    one = MG.from_rho(rho, mask, lanes=lanes)
    want = one.solve(f, tol=1e-9)[0]
    want_ap = one.apply(want)
    del one
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    print(f"dropped while in use on another stream {N}^3 lanes={lanes}", flush=True)
    mg = MG.from_rho(rho, mask, lanes=lanes)
    with torch.cuda.stream(side):
        p = mg.solve(f, tol=1e-9)[0]
        busy = pending(side)
        ap = mg.apply(p)
    sizes = [t.numel() for t in (mg.workspace, mg.lane_workspace) if t is not None]
    del mg
    filled = [torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda") for n in sizes]
    assert not busy.query()   # all that happened before the other stream went on
    torch.cuda.synchronize()
    assert torch.equal(p, want) and torch.equal(ap, want_ap)
    assert all(int(t.min()) == 0xFF for t in filled)


@pytest.mark.parametrize("changed", [False, True])
def test_destroy_waits(changed):
    """mg_destroy returns when the context's work is done, on the stream it was set up on or
    a later one; mg_release does not wait."""
    import ctypes
    from paper_1410_2240_amd import _lib
    lib = _lib.load()
    N = 16
    inp = fields.make("c2", N)
    rho, mask, p = dev(inp.rho), dev(inp.mask), dev(inp.f)
    ap = torch.empty_like(p)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    home, side = torch.cuda.current_stream(), torch.cuda.Stream()
    size = lib.mg_workspace_size(_lib.dims3(N), 0)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for end, done in ((lib.mg_release, False), (lib.mg_destroy, True)):
        print(f"{end.__name__}, stream changed: {changed}", flush=True)
        ctx = ctypes.c_void_p()
        assert lib.mg_setup_from_rho(ctypes.byref(ctx), ptr(ws), size, ptr(rho), ptr(mask), _lib.dims3(N), 1.0 / N, 0,
                                     ctypes.c_void_p(home.cuda_stream)) == 0, _lib.last_error()
        use = side if changed else home
        assert lib.mg_set_stream(ctx, ctypes.c_void_p(use.cuda_stream)) == 0
        with torch.cuda.stream(use):
            pending(use)
            assert lib.mg_apply(ctx, ptr(p), ptr(ap), 1) == 0
            event = use.record_event()
        end(ctx)
        assert event.query() == done
        torch.cuda.synchronize()


@pytest.mark.parametrize("handle", [None, 1, 2], ids=["null", "legacy", "per_thread"])
def test_special_stream_handles(handle):
    """The handles that name the default and the per-thread stream: setup, solves (one item,
    static scratch, a batch on lanes) and destruction, the bits of the null stream."""
    import ctypes
    from paper_1410_2240_amd import MG, _lib
    lib = _lib.load()
    N = 32
    inp = fields.make("c2", N)
    rho, mask, f = dev(inp.rho), dev(inp.mask), dev(fields.batch_rhs(inp.mask, 3))
    want = MG.from_rho(rho, mask).solve(f, tol=1e-9)[0]
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    empty = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    size, per = lib.mg_workspace_size(_lib.dims3(N), 0), lib.mg_lane_workspace_size(_lib.dims3(N), 0)
    ws, lane_ws = empty(size), empty(2 * per)
    p = [torch.zeros_like(f) for _ in range(3)]
    torch.cuda.synchronize()
    print(f"stream handle {handle}", flush=True)
    ctx = ctypes.c_void_p()
    assert lib.mg_setup_from_rho(ctypes.byref(ctx), ptr(ws), size, ptr(rho), ptr(mask), _lib.dims3(N), 1.0 / N, 0,
                                 ctypes.c_void_p(handle)) == 0, _lib.last_error()
    solve = lambda entry, x: entry(ctx, ptr(f), ptr(x), 3, 1e-9, 100, None, None, None)
    assert solve(lib.mg_solve, p[0]) == 0, _lib.last_error()
    assert solve(lib.mg_solve_static, p[1]) == 0, _lib.last_error()
    assert lib.mg_add_lanes(ctx, ptr(lane_ws), 2 * per, 2) == 0, _lib.last_error()
    assert lib.mg_set_stream(ctx, ctypes.c_void_p(handle)) == 0
    assert solve(lib.mg_solve, p[2]) == 0, _lib.last_error()
    lib.mg_destroy(ctx)
    assert all(torch.equal(x, want) for x in p)
