"""The propagation calls captured into a HIP graph (torch.cuda.CUDAGraph) and replayed.

After one call with the same parameters has allocated the context's scratch and tables,
a call enqueues kernels only, so it can be captured. Each replay is checked bit for bit
against an eager call on the replay's input, with other eager work on the device
between the replays."""
import sys

import numpy as np
import pytest

from paper_1107_5578_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    from paper_1107_5578_amd import cwo
    c = cwo.Context(0)
    yield c
    c.close()


def note(msg):
    print("[gpu-case] " + msg, flush=True)
    sys.stdout.flush()


def fields(n, count, seed):
    import torch
    return [torch.from_numpy(W.uniform_random_field(n, seed + k)).cuda() for k in range(count)]


@pytest.mark.parametrize("kind,n", [("asm", 512), ("fresnel", 256), ("asm", 2048)])
def test_plain_call_graph_replay(ctx, kind, n):
    import torch
    note("graph %s %d" % (kind, n))
    fn = ctx.asm if kind == "asm" else ctx.fresnel
    src = fields(n, 4, 900)
    u = src[0].clone()
    out = torch.empty_like(u)
    fn(u, 8e-6, 8e-6, 532e-9, 0.2, out=out)  # allocates scratch and tables
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn(u, 8e-6, 8e-6, 532e-9, 0.2, out=out)
    other = fields(n, 1, 77)[0]
    for rep, f in enumerate(src):
        u.copy_(f)
        g.replay()
        fn(other, 8e-6, 8e-6, 532e-9, 0.3)  # eager work between replays
        torch.cuda.synchronize()
        ref = fn(f, 8e-6, 8e-6, 532e-9, 0.2)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), rep


def test_zstack_graph_replay(ctx):
    import torch
    n = 512
    zs = list(W.zstack_distances(16, 0.05, 0.2))
    src = fields(n, 3, 910)
    u = src[0].clone()
    out = torch.empty((len(zs), n, n), dtype=torch.complex64, device="cuda")
    ctx.zstack(u, zs, 4e-6, 4e-6, 633e-9, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.zstack(u, zs, 4e-6, 4e-6, 633e-9, out=out)
    for rep, f in enumerate(src):
        u.copy_(f)
        g.replay()
        ctx.asm(f, 4e-6, 4e-6, 633e-9, 0.1)
        torch.cuda.synchronize()
        ref = ctx.zstack(f, zs, 4e-6, 4e-6, 633e-9)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), rep


def test_batch_graph_replay(ctx):
    import torch
    n = 256
    ins = fields(n, 8, 920)
    outs = [torch.empty_like(f) for f in ins]
    kw = dict(dx=8e-6, dy=8e-6, wavelength=532e-9, z=0.1)
    jobs = [("asm", f, o, kw) for f, o in zip(ins, outs)]
    ctx.batch(jobs)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.batch(jobs)
    for rep in range(3):
        for f in ins:
            f.mul_(1.5)
        g.replay()
        torch.cuda.synchronize()
        for f, o in zip(ins, outs):
            assert torch.equal(o, ctx.asm(f, 8e-6, 8e-6, 532e-9, 0.1)), rep


def test_point_light_source_and_fused_intensity_graph_replay(ctx):
    """The hologram sum and the fused-intensity propagation captured and replayed: each
    replay equals an eager call on the replay's inputs (eager calls between replays use no
    more points and no larger plane, so the captured scratch stays in place)."""
    import torch
    n, count = 256, 700
    clouds = [torch.from_numpy(W.pls_points(count, 950 + k, half_extent=2e-4)).cuda()
              for k in range(3)]
    pts = clouds[0].clone()
    holo = torch.empty((n, n), dtype=torch.float32, device="cuda")
    src = fields(n, 3, 960)
    u = src[0].clone()
    inten = torch.empty((n, n), dtype=torch.float32, device="cuda")
    args = (n, n, 4e-6, 4e-6, 633e-9, 1e-4, 0.0, 0.1)
    ctx.pls_cgh(pts, *args, out=holo)
    ctx.asm_intensity(u, 8e-6, 8e-6, 532e-9, 0.2, out=inten)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.pls_cgh(pts, *args, out=holo)
        ctx.asm_intensity(u, 8e-6, 8e-6, 532e-9, 0.2, out=inten)
    for rep in range(3):
        pts.copy_(clouds[rep])
        u.copy_(src[rep])
        g.replay()
        ctx.pls_cgh(clouds[(rep + 1) % 3][: count // 2].contiguous(), *args)  # eager, fewer points
        ctx.asm(src[(rep + 1) % 3], 8e-6, 8e-6, 532e-9, 0.3)
        torch.cuda.synchronize()
        ref_h = ctx.pls_cgh(clouds[rep], *args)
        ref_i = ctx.asm_intensity(src[rep], 8e-6, 8e-6, 532e-9, 0.2)
        torch.cuda.synchronize()
        assert torch.equal(holo, ref_h), rep
        assert torch.equal(inten, ref_i), rep


@pytest.mark.parametrize("first", [(2048, 2048, 4596, False), (64, 48, 3000, True)])
def test_point_light_source_graph_survives_smaller_holograms(first):
    """A hologram sum captured, then eager sums of no more points on other sizes that are summed
    in other numbers of point ranges (fewer pixels take more of them): the captured records and
    partial sums stay where they are, so every replay still equals the eager call."""
    import torch
    from paper_1107_5578_amd import cwo
    c = cwo.Context(0)
    nx, ny, count, field = first

    def run(t, nx, ny, field, out=None):
        fn = c.pls_field if field else c.pls_cgh
        return fn(t, nx, ny, 4e-6, 4e-6, 633e-9, 1e-4, 0.0, 0.1, out=out)

    clouds = [torch.from_numpy(W.pls_points(count, 970 + k, half_extent=2e-4)).cuda()
              for k in range(2)]
    pts = clouds[0].clone()
    out = run(pts, nx, ny, field)  # allocates
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(pts, nx, ny, field, out)
    for rep, (sx, sy, n, f) in enumerate([(512, 512, 4000, False), (256, 256, 2000, True),
                                          (1038, 496, 4596, False), (64, 64, 149, False)]):
        n = min(n, count)
        note("graph pls %dx%d, eager %dx%d points=%d field=%s" % (nx, ny, sx, sy, n, f))
        small = run(clouds[1][:n].contiguous(), sx, sy, f)
        pts.copy_(clouds[rep % 2])
        g.replay()
        torch.cuda.synchronize()
        ref = run(clouds[rep % 2], nx, ny, field)
        again = run(clouds[1][:n].contiguous(), sx, sy, f)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), rep
        assert torch.equal(small, again), rep
    c.close()


def test_first_partial_sums_beside_a_capture():
    """A plane is captured while a hologram of few pixels, the first to want partial sums, is
    summed on another stream: the graph is whole and the hologram right."""
    import torch
    from paper_1107_5578_amd import cwo
    note("pls beside a capture")
    planes, sums = cwo.Context(0), cwo.Context(0)
    src = fields(256, 3, 980)
    u, out = src[0].clone(), torch.empty_like(src[0])
    planes.asm(u, 8e-6, 8e-6, 532e-9, 0.2, out=out)
    pts = torch.from_numpy(W.pls_points(4000, 981, half_extent=2e-4)).cuda()
    args = (4e-6, 4e-6, 633e-9, 1e-4, 0.0, 0.1)
    sums.pls_cgh(pts[:100].contiguous(), 2048, 2048, *args)  # records for fewer points
    sums.pls_cgh(pts, 2048, 2048, *args)                     # one range
    held = sums.memory_held()
    holo = torch.empty((256, 256), device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        planes.asm(u, 8e-6, 8e-6, 532e-9, 0.2, out=out)
        sums.pls_cgh(pts, 256, 256, *args, out=holo, stream=side)
    torch.cuda.synchronize()
    assert sums.memory_held() == held + (64 << 20)
    for rep, f in enumerate(src):
        u.copy_(f)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, planes.asm(f, 8e-6, 8e-6, 532e-9, 0.2)), rep
    assert torch.equal(holo, sums.pls_cgh(pts, 256, 256, *args))
    planes.close()
    sums.close()
