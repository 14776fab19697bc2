"""The ways a sweep can visit a region give the same bits: only the rounds that can
change something, every round taken for live, whole pages streamed inside the
one-launch sweep, and the kernel that only streams.  A warm solve is made to take
one of them through the words its workspace holds (the head word of each region's
live bits, the last word of the signature).  And: which solves, warm starts and batches
stream."""
import numpy as np
import pytest
import torch

import oracle
import paper_1503_03492_amd as smre

pytestmark = pytest.mark.gpu

ALL_LIVE, STREAM = 1, 20  # head words (0: by the live bits; STREAM: for 19 sweeps more)


@pytest.fixture(scope="module")
def ctx():
    c = smre.Context(0)
    yield c
    c.close()


def heads(ws, H, W, R, nsides):
    """View of the regions' head words, [row][column]."""
    words = ws.view(torch.int32)
    qbytes = int(ws.view(torch.int64)[(ws.numel() - 256) // 8 + 6])
    nry, nrx, stride = -(-H // R), -(-W // R), 4 + nsides * R * R // 32
    at = (qbytes - -(-nry * nrx * stride * 4 // 256) * 256) // 4
    return words[at:at + nry * nrx * stride].view(nry, nrx, stride)[:, :, 0]


def signature_tail(ws):
    return ws.view(torch.int64)[(ws.numel() - 256) // 8 + 7:(ws.numel() - 256) // 8 + 8]


def first_sweeps(ctx, x0, sides, n, **kw):
    """n sweeps from zero increments: the workspace they leave."""
    H, W = x0.shape
    o = smre.ProjectOptions(tol=0, max_sweeps=n, **kw)
    r2 = smre.chi2_bounds(sides)
    dt = smre.F64 if x0.dtype == torch.float64 else smre.F32
    size = ctx.workspace_size(dt, H, W, sides, r2, o)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    ctx.project(x0.clone(), sides, r2, o, workspace=ws)
    signature_tail(ws)[0] = 0  # (so few sweeps keep their live bits)
    return ws


def go_on(ctx, x0, sides, n, ws, **kw):
    x = x0.clone()
    ctx.project(x, sides, smre.chi2_bounds(sides), tol=0, max_sweeps=n, warm=True, workspace=ws,
                **kw)
    return x


def image(H, W, dtype, seed=1):
    """Quiet on the left, most windows outside their bounds on the right."""
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(H, W, generator=g, dtype=torch.float64)
    x[:, :W // 2] *= 0.1
    x[:, W // 2:] = 4.0 * x[:, W // 2:] + 3.0
    x[H // 2, W // 5] = 9.0
    return x.to(dtype).cuda()


@pytest.mark.parametrize("dtype,inc,kahan", [
    (torch.float32, smre.INC_SAME, True), (torch.float32, smre.INC_SAME, False),
    (torch.float32, smre.INC_BF16, True), (torch.float32, smre.INC_BF16, False),
    (torch.float64, smre.INC_SAME, True)])
@pytest.mark.parametrize("R,H,W,sides", [
    (8, 40, 53, list(range(1, 10))), (16, 61, 70, list(range(1, 10))),
    (16, 64, 95, list(range(1, 17))), (32, 75, 101, [1, 2, 5, 8, 9, 16, 17, 24, 31, 32])])
def test_every_way_gives_the_same_bits(ctx, dtype, inc, kahan, R, H, W, sides):
    kw = dict(region=R, inc=inc, kahan=kahan)
    x0 = image(H, W, dtype)
    ws = first_sweeps(ctx, x0, sides, 2, **kw)
    got = []
    for way in ("visit", "all live", "stream", "stream_phase"):
        w = ws.clone()
        h = heads(w, H, W, R, len(sides))
        if way == "visit":
            h.clamp_(max=ALL_LIVE)  # (the live bits of a region that streamed are stale)
        elif way == "stream_phase":
            signature_tail(w)[0] = 1
        else:
            h[:] = ALL_LIVE if way == "all live" else STREAM
        got.append(go_on(ctx, x0, sides, 2, w, **kw))
        # and once more from what that solve left
        got.append(go_on(ctx, x0, sides, 1, w, **kw))
    for i in range(2, len(got)):
        assert torch.equal(got[i], got[i % 2]), i


def test_streamed_region_waits_for_long_jobs_around_it(ctx):
    # the region of the last colour streams and waits for three regions of earlier
    # colours, one after the other, that visit every one of their 19617 rounds
    H = W = 95
    sides = list(range(1, 33))
    x0 = image(H, W, torch.float64) + 5.0
    ws = first_sweeps(ctx, x0, sides, 1, region=32)
    want = ws.clone()
    heads(want, H, W, 32, len(sides)).clamp_(max=ALL_LIVE)
    h = heads(ws, H, W, 32, len(sides))
    h[:2, :2] = ALL_LIVE
    h[1, 1] = STREAM
    assert torch.equal(go_on(ctx, x0, sides, 1, ws, region=32),
                       go_on(ctx, x0, sides, 1, want, region=32))


def test_a_sweep_of_equal_jobs_takes_about_four_of_them(ctx):
    # 256 regions of each colour, all streamed: one launch that orders them itself
    # against four launches of the streaming kernel (measured 347 and 323 us; 507
    # when a workgroup could hold two regions of one colour)
    H = W = 512
    sides = list(range(1, 9))
    x0 = image(H, W, torch.float32)
    ws = first_sweeps(ctx, x0, sides, 2, region=16)
    us = []
    for one_launch in (True, False):
        best = 1e9
        for _ in range(8):
            w = ws.clone()
            if one_launch:
                heads(w, H, W, 16, len(sides))[:] = STREAM
            else:
                signature_tail(w)[0] = 1
            ctx.set_timing(True)
            _, rep = ctx.project(x0.clone(), sides, smre.chi2_bounds(sides), tol=0, max_sweeps=1,
                                 warm=True, workspace=w, region=16)
            ctx.set_timing(False)
            best = min(best, rep["kernel_ms"] * 1e3)
        us.append(best)
    assert us[0] <= 1.3 * us[1], us


def solved(ctx, x0, sides, **kw):
    """The workspace a cold solve leaves, and its report."""
    o = smre.ProjectOptions(**kw)
    r2 = smre.chi2_bounds(sides)
    ws = torch.zeros(ctx.workspace_size(smre.F32, *x0.shape, sides, r2, o), dtype=torch.uint8,
                     device="cuda")
    _, rep = ctx.project(x0.clone(), sides, r2, o, workspace=ws)
    return ws, rep


def dense_corner(n, k):
    g = torch.Generator().manual_seed(3)
    x = 0.02 * torch.randn(n, n, generator=g, dtype=torch.float64)
    x[:k, :k] += 40.0 * torch.randn(k, k, generator=g, dtype=torch.float64)
    return x.float().cuda()


@pytest.mark.parametrize("every", [1, 10])
def test_a_dense_corner_does_not_stream_the_whole_image(ctx, every):
    # about 16 of 256 regions stream: far from the third at which the solve goes over,
    # however many sweeps lie between two checks
    ws, _ = solved(ctx, dense_corner(256, 64), list(range(1, 9)), tol=1e-12, max_sweeps=25,
                   check_every=every, region=16)
    assert int((heads(ws, 256, 256, 16, 8) > 1).sum()) > 0
    assert int(signature_tail(ws)[0]) == 0


@pytest.mark.parametrize("tol,every", [(0, 1), (1e-12, 1), (1e-12, 7)])
def test_a_dense_image_goes_over_to_streaming(ctx, tol, every):
    ws, _ = solved(ctx, dense_corner(128, 128), list(range(1, 9)), tol=tol, max_sweeps=20,
                   check_every=every, region=16)
    assert int(signature_tail(ws)[0]) == 1


@pytest.mark.parametrize("amp,streams", [(1.0, 1), (0.01, 0)])
def test_a_short_solve_hands_on_that_its_image_streams(ctx, amp, streams):
    # (a chain of warm solves of one to three sweeps, as in an ADMM loop)
    ws, _ = solved(ctx, amp * dense_corner(128, 128), list(range(1, 9)), tol=1e-12, max_sweeps=1,
                   region=16)
    assert int(signature_tail(ws)[0]) == streams


@pytest.mark.parametrize("n,sides,amp,streams", [
    (128, list(range(1, 9)), 1.0, True),       # 239 rounds a region
    (33, [2, 3, 8], 1.0, True),                # fewer tiles than the sample holds
    (128, list(range(1, 9)), 0.02, False),     # within the bounds
    (128, list(range(1, 11)), 1.0, False),     # 420 rounds a region: visiting is as good
])
def test_a_dense_input_streams_from_the_first_sweep(ctx, n, sides, amp, streams):
    ws, _ = solved(ctx, amp * dense_corner(n, n), sides, tol=0, max_sweeps=1, region=16)
    # (a sweep that visits leaves every region's head word at 32 or at 0)
    visited = int(heads(ws, n, n, 16, len(sides)).max()) > 0 or int(signature_tail(ws)[0]) == 0
    assert visited != streams


@pytest.mark.parametrize("use_graph", [True, False])
@pytest.mark.parametrize("amps", [(1.0, 1.0, 1.0), (1.0, 0.05, 0.02), (0.1, 0.075, 1.0)])
def test_dense_batch_equals_single(ctx, amps, use_graph):
    # all images streaming, some, and some that go over to it while others are visited
    sides = list(range(1, 9))
    r2 = smre.chi2_bounds(sides)
    xs0 = [a * dense_corner(n, n) for a, n in zip(amps, (70, 96, 48))]
    xs = [x.clone() for x in xs0]
    _, reps = ctx.project_batch(xs, sides, r2, tol=1e-4, max_sweeps=40, region=16,
                                use_graph=use_graph)
    for x0, x, rep in zip(xs0, xs, reps):
        y = x0.clone()
        _, one = ctx.project(y, sides, r2, tol=1e-4, max_sweeps=40, region=16)
        assert torch.equal(x, y)
        assert rep["sweeps"] == one["sweeps"] and rep["converged"] == one["converged"]


@pytest.mark.parametrize("amp,streams", [(4.0, 1), (0.6, 0)])
def test_warm_start_after_either_kind_of_solve(ctx, amp, streams):
    # eight sweeps that go over to streaming on the way (half of the image dense), or
    # stay with visiting, then a warm solve of a moved image from the increments they leave
    H, W, sides, R = 70, 61, list(range(1, 9)), 16
    r2 = smre.chi2_bounds(sides)
    rng = np.random.default_rng(8)
    xa = amp * rng.standard_normal((H, W))
    xa[:, 32:] *= 0.1
    xa[20:24, 40:44] += 3.0
    xb = xa + 0.05 * rng.standard_normal((H, W))
    o = smre.ProjectOptions(tol=0, max_sweeps=8, region=R)
    ws = torch.zeros(ctx.workspace_size(smre.F64, H, W, sides, r2, o), dtype=torch.uint8,
                     device="cuda")
    ctx.project(torch.from_numpy(xa).cuda(), sides, r2, o, workspace=ws)
    assert int(signature_tail(ws)[0]) == streams
    x = torch.from_numpy(xb).cuda()
    ctx.project(x, sides, r2, tol=0, max_sweeps=3, region=R, warm=True, workspace=ws)
    _, _, _, ia = oracle.dykstra(xa, sides, r2, tol=0, max_sweeps=8, order=oracle.ORDER_REGION,
                                 region=R, want_incs=True)
    ref, _, _ = oracle.dykstra(xb, sides, r2, tol=0, max_sweeps=3, order=oracle.ORDER_REGION,
                               region=R, incs0=ia)
    # a few hundred roundings of 1e-16 a sweep
    assert np.max(np.abs(x.cpu().numpy() - ref)) <= 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("H,W", [(1100, 1070), (3000, 41), (7, 5000)])
@pytest.mark.parametrize("every", [1, 2])
def test_the_streaming_solve_reports_its_largest_change(ctx, H, W, every):
    # (more tiles than the check has workgroups, and images narrower than a tile)
    sides, r2 = [1, 2, 4], smre.chi2_bounds([1, 2, 4])
    x0 = dense_corner(max(H, W), min(H, W))[:H, :W].contiguous() if H * W < 10 ** 6 else \
        3.0 * torch.randn(H, W, generator=torch.Generator().manual_seed(6)).cuda()
    xs = []
    for sweeps in (3, 4):
        xs.append(x0.clone())
        ctx.project(xs[-1], sides, r2, tol=0, max_sweeps=sweeps, region=16)
    x = x0.clone()
    _, rep = ctx.project(x, sides, r2, tol=1e-12, max_sweeps=4, check_every=every, region=16)
    assert torch.equal(x, xs[1])
    assert rep["last_delta"] == float((xs[1].double() - xs[0].double()).abs().max())
