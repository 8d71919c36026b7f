"""Planes at the edges of the row and column passes' layouts: the narrowest and shortest tiled
planes, the split form of 8192 with few rows or columns, and the passes on each side of a
change of form, against the FP64 oracle. Bound: relative L2 <= 1e-5, as for every FP32 plane
(four transforms of about eps32 * log2(M) each and a phase rounded to 2^-24 revolution)."""
import numpy as np
import pytest
import torch

from oracle import diffraction as D
from oracle import shifted_fresnel as SF
from paper_1107_5578_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def gpu():
    if not torch.cuda.is_available():  # (initialises torch's runtime before the library loads)
        pytest.fail("GPU tests need a ROCm device")

SHAPES = [(128, 16), (256, 16), (256, 32), (16, 256), (512, 16), (1024, 16), (2048, 16),
          (4096, 16), (4096, 32), (256, 4096), (16, 4096), (4096, 4096)]


@pytest.mark.parametrize("kind", [D.ASM, D.FRESNEL])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_plane_edges(kind, nx, ny):
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    u = W.uniform_random_field(nx, nx + 3 * ny, ny=ny)
    dx, lam, z = 8e-6, 532e-9, 0.03
    print("[gpu-case] plane %s %dx%d" % (kind, nx, ny), flush=True)
    t = torch.from_numpy(u).cuda()
    y = (ctx.asm if kind == D.ASM else ctx.fresnel)(t, dx, dx, lam, z).cpu().numpy()
    assert D.rel_l2(y, D.propagate(u, kind, dx, dx, lam, z)) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("nx,ny", [(64, 32), (256, 16), (16, 256), (512, 64), (2048, 16), (4096, 16)])
def test_shifted_fresnel_edges(nx, ny):
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    u = W.uniform_random_field(nx, nx + 5 * ny, ny=ny)
    args = (8e-6, 8e-6, 6e-6, 7e-6, 532e-9, 0.2, 0.0, 0.0, 2e-4, -1e-4)
    print("[gpu-case] shifted fresnel %dx%d" % (nx, ny), flush=True)
    y = ctx.fresnel_shifted(torch.from_numpy(u).cuda(), *args).cpu().numpy()
    assert D.rel_l2(y, SF.propagate(u, *args)) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("n,nz", [(16, 3), (64, 1), (128, 64), (256, 65), (512, 2)])
def test_zstack_groups(n, nz):
    """Planes per launch cut into groups (and a second launch beyond 64): every plane equals
    the single propagation to rounding."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    t = torch.from_numpy(W.speckle_field(n, n + nz)).cuda()
    z = np.linspace(0.05, 0.2, nz)
    print("[gpu-case] zstack %d x%d" % (n, nz), flush=True)
    s = ctx.zstack(t, z, 8e-6, 8e-6, 532e-9)
    for k in sorted({0, nz // 2, nz - 1}):
        one = ctx.asm(t, 8e-6, 8e-6, 532e-9, float(z[k]))
        assert D.rel_l2(s[k].cpu().numpy(), one.cpu().numpy().astype(np.complex128)) <= 1e-6
    ctx.close()


@pytest.mark.parametrize("n,count", [(256, 3), (1024, 16), (2048, 3)])
def test_batch_beyond_the_caches(n, count):
    """Batches on both sides of the size from which results are stored past the caches: each
    result equals the single propagation (the same transforms, so the bound of two FP32
    evaluations), also where the output is the input."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    us = [torch.from_numpy(W.uniform_random_field(n, n + k)).cuda() for k in range(count)]
    kw = dict(dx=8e-6, wavelength=532e-9, z=0.03)
    print("[gpu-case] batch %d x%d" % (n, count), flush=True)
    one = [ctx.asm(u, 8e-6, None, 532e-9, 0.03) for u in us]
    ctx.batch([("asm", u, u, kw) for u in us])
    for a, b in zip(us, one):
        assert D.rel_l2(a.cpu().numpy(), b.cpu().numpy()) <= 2e-6
    ctx.close()


@pytest.mark.parametrize("nx,ny", [(16, 2048), (2048, 16), (16, 4096), (4096, 16), (64, 16), (16, 64), (512, 1024)])
def test_zstack_widths(nx, ny):
    """The column groups of z-stack planes follow the column length alone: planes much wider or
    taller than square equal the single propagation to rounding."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    t = torch.from_numpy(W.uniform_random_field(nx, nx + 7 * ny, ny=ny)).cuda()
    z = np.linspace(0.02, 0.05, 5)
    print("[gpu-case] zstack widths %dx%d" % (nx, ny), flush=True)
    for kind, single in (("asm", ctx.asm), ("fresnel", ctx.fresnel)):
        s = ctx.zstack(t, z, 8e-6, 8e-6, 532e-9, kind=kind)
        for k in (0, 4):
            one = single(t, 8e-6, 8e-6, 532e-9, float(z[k]))
            assert D.rel_l2(s[k].cpu().numpy(), one.cpu().numpy().astype(np.complex128)) <= 1e-6
    ctx.close()


@pytest.mark.parametrize("n,count", [(256, 2), (256, 64), (512, 31), (512, 32), (1024, 2)])
def test_batch_layouts(n, count):
    """Batches on both sides of the change from tiled to row-major planes against single
    propagations (the bound of two FP32 evaluations)."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    us = [torch.from_numpy(W.uniform_random_field(n, n + k)).cuda() for k in range(count)]
    os = [torch.empty_like(u) for u in us]
    kind = lambda k: "fresnel" if k % 3 == 1 else "asm"
    print("[gpu-case] batch layouts %d x%d" % (n, count), flush=True)
    ctx.batch([(kind(k), u, o, dict(dx=8e-6, wavelength=532e-9, z=0.03 + 0.01 * k))
               for k, (u, o) in enumerate(zip(us, os))])
    for k in (0, 1, count // 2, count - 1):
        one = (ctx.fresnel if kind(k) == "fresnel" else ctx.asm)(us[k], 8e-6, None, 532e-9, 0.03 + 0.01 * k)
        assert D.rel_l2(os[k].cpu().numpy(), one.cpu().numpy().astype(np.complex128)) <= 2e-6
    ctx.close()


@pytest.mark.parametrize("nx,ny,at", [(16, 16, 0), (16, 16, 255), (512, 64, 32767), (2048, 1024, 2097151),
                                      (1024, 1024, 700001), (2048, 2048, 4194303)])
def test_range_of_fp16_storage(nx, ny, at):
    """The largest value anywhere in the field sets the power-of-two scale: a spike of 3e4 alone
    in a field of 1e-3, at the first, the last and inner places, keeps the FP16 bound 3e-3."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    u = (1e-3 * W.uniform_random_field(nx, nx + ny, ny=ny)).astype(np.complex64)
    u.reshape(-1)[at] = 3e4
    print("[gpu-case] fp16 range %dx%d at %d" % (nx, ny, at), flush=True)
    t = torch.from_numpy(u).cuda()
    y = ctx.asm(t, 8e-6, None, 532e-9, 0.03, precision="f16").cpu().numpy()
    assert np.isfinite(y).all()
    assert D.rel_l2(y, ctx.asm(t, 8e-6, None, 532e-9, 0.03).cpu().numpy().astype(np.complex128)) <= 3e-3
    ctx.close()


@pytest.mark.parametrize("nx,ny", [(16, 16), (64, 32), (512, 16), (16, 1024), (4096, 32), (1024, 1024), (256, 4096)])
def test_gs_error_sums(nx, ny):
    """E_0 for few and many partial sums of the rows and of the target (and not a multiple of
    the threads that add them): a field off by 1e-5 of its norm moves E by at most that over the
    target's norm."""
    from oracle import gs as G
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    u = W.uniform_random_field(nx, nx + 11 * ny, ny=ny)
    a2 = np.abs(W.uniform_random_field(nx, nx + 13 * ny, ny=ny)).astype(np.float32)
    a1 = np.ones_like(a2)
    print("[gpu-case] gs errors %dx%d" % (nx, ny), flush=True)
    e = ctx.gs(torch.from_numpy(u).cuda(), torch.from_numpy(a1).cuda(), torch.from_numpy(a2).cuda(),
               8e-6, None, 532e-9, 0.03, iterations=1).cpu().numpy()[0]
    v = D.propagate(u, D.ASM, 8e-6, 8e-6, 532e-9, 0.03)
    want = G.error(v, a2)
    assert abs(e - want) <= 1e-5 * np.linalg.norm(v) / np.linalg.norm(a2) + 1e-6 * want
    ctx.close()


@pytest.mark.parametrize("nx,ny", [(4096, 16), (4096, 64), (2048, 32), (256, 16), (128, 64)])
def test_gs_field_and_errors(nx, ny):
    """Three iterations of the row kernel's forms (split rows of 8192, whole tiled rows, row-major
    rows) against the oracle: the field and every E_k. Six propagations, each within 5e-7 of its
    norm, and constraints that enlarge an error by the ratio of amplitudes (a few) stay below 1e-5."""
    from oracle import gs as G
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    y, x = np.mgrid[0:ny, 0:nx].astype(np.float64)
    a1 = (0.9 + 0.1 * np.cos(2e-3 * x + 0.3 * y)).astype(np.float32)
    a2 = (0.75 + 0.25 * np.cos(5e-3 * x - 0.2 * y)).astype(np.float32)
    u = (a1 * np.exp(0.3j * np.cos(4e-3 * x + 0.1 * y))).astype(np.complex64)
    print("[gpu-case] gs field %dx%d" % (nx, ny), flush=True)
    v = torch.from_numpy(u).cuda()
    e = ctx.gs(v, torch.from_numpy(a1).cuda(), torch.from_numpy(a2).cuda(), 8e-6, None, 532e-9, 0.01,
               iterations=3).cpu().numpy()
    r = u
    for k in range(3):
        r, want = G.iteration(r, a1, a2, 8e-6, 532e-9, 0.01)
        assert abs(e[k] - want) <= 1e-5
    assert D.rel_l2(v.cpu().numpy(), r) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("nx,ny,count", [(256, 4096, 8), (512, 2048, 9), (512, 64, 64), (256, 512, 33)])
def test_batch_of_rectangles(nx, ny, count):
    """Batches of 128 MiB of planes and more of narrow, tall and flat fields equal the single
    calls bit for bit."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    us = [torch.from_numpy(W.uniform_random_field(nx, nx + k, ny=ny)).cuda() for k in range(count)]
    os = [torch.empty_like(u) for u in us]
    print("[gpu-case] batch %dx%d x%d" % (nx, ny, count), flush=True)
    ctx.batch([("asm", u, o, dict(dx=8e-6, wavelength=532e-9, z=0.03)) for u, o in zip(us, os)])
    for k in (0, count // 2, count - 1):
        assert torch.equal(os[k], ctx.asm(us[k], 8e-6, None, 532e-9, 0.03))
    ctx.close()


@pytest.mark.parametrize("nx,ny", [(16, 16), (128, 64), (16, 256), (256, 16)])
def test_noalloc_short_transforms(nx, ny):
    """Transforms below 512 points take their factors from the end of the tables, which the
    static scratch holds as well."""
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    t = torch.from_numpy(W.uniform_random_field(nx, nx + 17 * ny, ny=ny)).cuda()
    out = torch.empty_like(t)
    print("[gpu-case] noalloc %dx%d" % (nx, ny), flush=True)
    ctx.asm_noalloc(t, 8e-6, None, 532e-9, 0.03, out=out)
    assert torch.equal(out, ctx.asm(t, 8e-6, None, 532e-9, 0.03))
    ctx.close()
