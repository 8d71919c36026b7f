"""How far complex64 results are from the FP64 oracle, against what the library's first arithmetic
gives on the same inputs: every value twiddled and then transformed by 4 x 4 points, transfer
functions from separately reduced phases or tabulated factors. The bounds are its relative L2
errors (means of three inputs, rounded up in the third digit), measured on an MI355X; a faster
arithmetic may not be further off."""
import numpy as np
import pytest
import torch

from oracle import diffraction as D
from oracle import fresnel_fourier as FF
from oracle import gs as G
from oracle import pls as PL
from oracle import shifted_asm as SA
from oracle import shifted_fresnel as SF
from paper_1107_5578_amd import workloads as W

pytestmark = pytest.mark.gpu

LAM = 532e-9
BOUNDS = {
    ('asm', 64, 64): 2.81e-07, ('asm', 128, 128): 2.85e-07, ('asm', 256, 256): 3.29e-07,
    ('asm', 1024, 512): 3.22e-07, ('asm', 2048, 256): 2.92e-07, ('asm', 4096, 64): 2.76e-07,
    ('exact', 64, 64): 2.10e-07, ('exact', 128, 128): 2.29e-07, ('exact', 256, 256): 2.58e-07,
    ('exact', 1024, 512): 2.50e-07,
    ('fresnel', 64, 64): 1.88e-07, ('fresnel', 128, 128): 2.06e-07,
    ('fresnel', 256, 256): 2.48e-07, ('fresnel', 1024, 512): 2.55e-07,
    ('fresnel', 4096, 64): 2.51e-07,
    ('shifted', 64, 64): 2.83e-07, ('shifted', 128, 128): 2.96e-07,
    ('shifted', 256, 256): 3.42e-07, ('shifted', 1024, 512): 3.32e-07,
    ('sfresnel', 64, 64): 2.27e-07, ('sfresnel', 128, 128): 2.28e-07,
    ('sfresnel', 256, 256): 2.51e-07, ('sfresnel', 1024, 512): 2.68e-07,
    ('zstack', 64, 64): 2.26e-07, ('zstack', 128, 128): 2.53e-07, ('zstack', 256, 256): 2.86e-07,
    ('zstack', 1024, 512): 2.47e-07,
    ('zfresnel', 64, 64): 1.88e-07, ('zfresnel', 128, 128): 2.15e-07,
    ('zfresnel', 256, 256): 2.45e-07, ('zfresnel', 1024, 512): 2.56e-07,
    ('fourier', 16, 16): 1.09e-07, ('fourier', 64, 64): 1.37e-07, ('fourier', 256, 256): 1.56e-07,
    ('fourier', 512, 1024): 1.73e-07, ('fourier', 4096, 64): 1.68e-07,
    ('gs', 64, 64): 2.85e-07, ('gs', 256, 256): 2.14e-07, ('gs', 512, 512): 2.19e-07,
    ('pls150', 300, 200): 2.40e-07,
    ('pls256', 300, 200): 3.02e-07,
    ('pls260', 300, 200): 3.05e-07,
    ('pls300', 300, 200): 3.25e-07,
    ('pls383', 300, 200): 3.65e-07,
    ('pls384', 300, 200): 3.66e-07,
    ('pls600', 300, 200): 3.95e-07,
    ('pls2000', 300, 200): 4.15e-07,
}


@pytest.fixture(autouse=True, scope="module")
def gpu():
    if not torch.cuda.is_available():  # (initialises torch's runtime before the library loads)
        pytest.fail("GPU tests need a ROCm device")


def _results(ctx, op, nx, ny, seed):
    """The library's result and the oracle's for one input."""
    u = W.uniform_random_field(nx, 1000 * seed + nx + 3 * ny, ny=ny)
    t = torch.from_numpy(u).cuda()
    if op == "asm":
        return ctx.asm(t, 8e-6, None, LAM, 0.2), D.asm(u, 8e-6, None, LAM, 0.2)
    if op == "exact":  # a pitch of two wavelengths: beyond the series form
        return ctx.asm(t, 1e-6, None, LAM, 2e-3), D.asm(u, 1e-6, None, LAM, 2e-3)
    if op == "fresnel":
        return ctx.fresnel(t, 8e-6, None, LAM, 0.2), D.fresnel(u, 8e-6, None, LAM, 0.2)
    if op == "shifted":
        a = (8e-6, 8e-6, LAM, 0.2, 1e-4, -2e-4)
        return ctx.asm_shifted(t, *a), SA.propagate(u, *a)
    if op == "sfresnel":
        a = (8e-6, 8e-6, 12e-6, 12e-6, LAM, 0.5, 0.0, 0.0, 2e-3, -1e-3)
        return ctx.fresnel_shifted(t, *a), SF.propagate(u, *a)
    if op == "fourier":
        return ctx.fresnel_fourier(t, 8e-6, None, LAM, 0.5), FF.propagate(u, 8e-6, None, LAM, 0.5)
    if op == "zstack":
        z = [0.05, 0.11, 0.2]
        return (ctx.zstack(t, z, 8e-6, None, LAM)[1], D.asm(u, 8e-6, None, LAM, z[1]))
    if op == "zfresnel":
        z = [0.05, 0.11, 0.2]
        return (ctx.zstack(t, z, 8e-6, None, LAM, kind="fresnel")[1],
                D.fresnel(u, 8e-6, None, LAM, z[1]))
    if op == "gs":  # a smooth beam and target, three iterations
        y, x = np.mgrid[0:ny, 0:nx] / float(ny)
        a1 = (0.9 + 0.1 * np.cos(7 * x + seed) * np.cos(5 * y)).astype(np.float32)
        a2 = (0.75 + 0.25 * np.cos(4 * x) * np.cos(9 * y + seed)).astype(np.float32)
        u = (a1 * np.exp(0.3j * np.cos(6 * x - 8 * y))).astype(np.complex64)
        v = torch.from_numpy(u).cuda()
        ctx.gs(v, torch.from_numpy(a1).cuda(), torch.from_numpy(a2).cuda(), 8e-6, None, LAM, 0.08,
               iterations=3)
        r = u
        for _ in range(3):
            r = G.iteration(r, a1, a2, 8e-6, LAM, 0.08)[0]
        return v, r
    pts = W.pls_points(int(op[3:]), seed, half_extent=4e-3)
    a = (nx, ny, 4e-6, 4e-6, 633e-9, 10e-3, -2e-3, 0.2)
    return ctx.pls_cgh(torch.from_numpy(pts).cuda(), *a), PL.cgh(pts, *a)


def mean_error(op, nx, ny):
    from paper_1107_5578_amd import cwo
    ctx = cwo.Context(0)
    e = []
    for seed in (1, 2, 3):
        y, ref = _results(ctx, op, nx, ny, seed)
        y = y.cpu().numpy().astype(np.asarray(ref).dtype)
        e.append(float(np.linalg.norm((y - ref).ravel()) / np.linalg.norm(np.asarray(ref).ravel())))
    ctx.close()
    return sum(e) / len(e)


@pytest.mark.parametrize("op,nx,ny", list(BOUNDS))
def test_no_further_off_than_the_first_arithmetic(op, nx, ny):
    e = mean_error(op, nx, ny)
    print("[gpu-case] accuracy %s %dx%d: %.4e" % (op, nx, ny, e), flush=True)
    assert e <= BOUNDS[op, nx, ny]
