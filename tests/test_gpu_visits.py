"""The ways a sweep can visit a region, taken by warm solves through the words their
workspace holds (the head word of each region's live bits)."""
import pytest
import torch

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


def first_sweeps(ctx, x0, sides, n, **kw):
    """n sweeps from zero increments: the workspace they leave."""
    H, W = x0.shape
    o = smre.ProjectOptions(tol=0, max_sweeps=n, **kw)
    r2 = smre.chi2_bounds(sides)
    dt = smre.F64 if x0.dtype == torch.float64 else smre.F32
    size = ctx.workspace_size(dt, H, W, sides, r2, o)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    ctx.project(x0.clone(), sides, r2, o, workspace=ws)
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
