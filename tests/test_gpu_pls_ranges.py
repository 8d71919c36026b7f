"""Point-light-source sums where the kernel takes another branch: fewer or more points than
the finer phase is for (256), remainders of the 128-point sums and 256-point chunks, point
ranges summed apart (few pixels, many points), rows that are no multiple of a lane's, chunks
with a point too far in phase for the short form, and a budget without room for partial sums.

Bounds as in test_gpu_pls: a term is off by at most ~4e-7 |A_j| (2^-24 revolution of phase,
2.4e-7 rad, plus the hardware cosine's 1.3e-7), FP32 sums of 128 points add eps32 * sqrt(128)
of their size, so |I - I_ref| <= 1e-6 sum |A_j| and relative L2 <= 1e-5.
"""
import numpy as np
import pytest
import torch

from oracle import pls as PL
from paper_1107_5578_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def gpu():
    if not torch.cuda.is_available():  # (initialises torch's runtime before the library loads)
        pytest.fail("GPU tests need a ROCm device")


def _run(ctx, pts, args, field):
    t = torch.from_numpy(np.ascontiguousarray(pts, dtype=np.float32)).cuda()
    out = (ctx.pls_field if field else ctx.pls_cgh)(t, *args)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _check(y, pts, args, field):
    lam, oz = args[4], args[7]
    ref = (PL.field if field else PL.cgh)(pts, *args)
    scale = 1.0 / abs(lam * oz) if field else 1.0
    assert np.all(np.isfinite(y))
    assert np.abs(y - ref).max() <= 1e-6 * scale * float(np.abs(pts[:, 3]).sum())
    assert np.linalg.norm((y - ref).ravel()) <= 1e-5 * np.linalg.norm(ref.ravel())


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("nx,ny,count", [
    (64, 8, 255), (65, 9, 256), (63, 7, 257), (130, 33, 385), (70, 5, 4000), (400, 31, 129),
    (1030, 130, 300)])
def test_counts_and_sizes(field, nx, ny, count):
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    pts = W.pls_points(count, 31 + count, half_extent=2e-4)
    args = (nx, ny, 5e-6, 6e-6, 532e-9, 3e-5, -2e-5, 0.05)
    print("[gpu-case] pls field=%s %dx%d points=%d" % (field, nx, ny, count), flush=True)
    _check(_run(ctx, pts, args, field), pts, args, field)
    ctx.close()


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("far", [1, 300])
def test_far_phase_chunk(field, far):
    """Points 10 um from the plane: c r^2 is 5e5 to 2e6 revolutions, beyond the short form's
    2^18; only their chunks take the FP64 fraction."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    pts = W.pls_points(600, 77, half_extent=2e-4)
    args = (96, 40, 5e-6, 6e-6, 532e-9, 3e-3, -2e-3, 0.05)
    pts[:far, 2] = np.float32(1e-5 - 0.05)
    print("[gpu-case] pls far phase field=%s far=%d" % (field, far), flush=True)
    _check(_run(ctx, pts, args, field), pts, args, field)
    ctx.close()


def test_point_in_the_plane_is_not_finite():
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    pts = W.pls_points(300, 78, half_extent=2e-4)
    pts[150, 2] = -0.0625
    y = _run(ctx, pts, (64, 16, 5e-6, 5e-6, 532e-9, 0.0, 0.0, 0.0625), False)
    assert not np.isfinite(y).any()
    ctx.close()


def test_budget_without_room_for_partial_sums():
    """A context whose budget holds the point records and nothing more gives the same sums to
    FP64 order: one range instead of several."""
    from paper_1107_5578_amd import cwo
    pts = W.pls_points(4000, 79, half_extent=2e-4)
    args = (64, 16, 5e-6, 5e-6, 532e-9, 0.0, 0.0, 0.05)
    free, tight = cwo.Context(0), cwo.Context(0, 32 * 4000)
    a, b = _run(free, pts, args, False), _run(tight, pts, args, False)
    assert tight.memory_held() == 32 * 4000
    _check(a, pts, args, False)
    _check(b, pts, args, False)
    free.close()
    tight.close()


def test_partial_sums_take_no_room_of_a_budget():
    """A budget that holds a 2048 x 2048 plane and the point records, not partial sums beside
    them: the plane runs after holograms that would take several ranges, and their sums are
    one range's."""
    from paper_1107_5578_amd import cwo
    n, count, budget = 2048, 2000, 70 << 20
    ctx = cwo.Context(0, budget)
    pts = W.pls_points(count, 80, half_extent=2e-4)
    args = (256, 256, 5e-6, 5e-6, 532e-9, 0.0, 0.0, 0.05)
    print("[gpu-case] pls then a plane in %d MiB" % (budget >> 20), flush=True)
    y = _run(ctx, pts, args, True)
    assert ctx.memory_held() == 32 * count
    u = torch.from_numpy(W.uniform_random_field(n, 81)).cuda()
    plane = ctx.asm(u, 8e-6, 8e-6, 532e-9, 0.2)
    _check(_run(ctx, pts, args, False), pts, args, False)
    _check(y, pts, args, True)
    free = cwo.Context(0)
    assert torch.equal(plane, free.asm(u, 8e-6, 8e-6, 532e-9, 0.2))
    free.close()
    ctx.close()


@pytest.mark.parametrize("nx,ny,count", [(64, 48, 4000), (200, 150, 3000), (512, 64, 2500)])
@pytest.mark.parametrize("field", [False, True])
def test_point_ranges_are_taken(nx, ny, count, field):
    """Small holograms of many points allocate the partial sums (64 MiB, once): several ranges
    were summed, and the result is the oracle's."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    pts = W.pls_points(count, 90, half_extent=2e-4)
    args = (nx, ny, 5e-6, 6e-6, 532e-9, 0.0, 0.0, 0.05)
    print("[gpu-case] pls ranges %dx%d points=%d field=%s" % (nx, ny, count, field), flush=True)
    y = _run(ctx, pts, args, field)
    assert ctx.memory_held() == 32 * count + (64 << 20)
    _check(y, pts, args, field)
    ctx.close()
