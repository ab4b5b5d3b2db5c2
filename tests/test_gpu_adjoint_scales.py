"""GPU parity of the matrix-core adjoint with the FP64 oracle gradient where the scales of its operands
can go wrong: field gradients down to FP32's smallest numbers, wavelengths of very different strength,
field gradients with a mean (a spectrum with one frequency far above the rest) or with gratings
(single frequencies on the axes)."""
import math

import numpy as np
import pytest

import gwsgen
import oracle
from gwsgen import Grid
from gpu_util import problem, rel_l2, scene_to_torch, to_numpy

pytestmark = pytest.mark.gpu

# Per term the phase's FP32 roundings are 1.5e-6 at most (three of 2^-22 of a revolution), the
# polynomial and the fp16 pairs 1e-7 each; a sum weighted by m or m^2 may cancel to about a third of
# its terms' norm.  5e-6 bounds the normwise error of every gradient.
TOL = 5e-6
LAMBDAS = (638e-9, 520e-9, 450e-9, 570e-9)


@pytest.fixture(scope="module")
def ctx():
    import torch
    import paper_2505_06582_amd as gws
    assert torch.cuda.is_available()
    return gws.context(0)


def gradients(ctx, scene, grid, G, depth=True):
    """{name: (the library's, the oracle's for the library's own FP32 spectrum of G)}: the error of the sums
    alone, without the transform's, which is in proportion to the whole field gradient."""
    import torch
    Gt = torch.from_numpy(np.ascontiguousarray(G, dtype=np.complex64)).cuda()
    got = ctx.backward(problem(grid), scene_to_torch(scene), Gt, want_depth=depth)
    spec = to_numpy(ctx.dft2d(Gt, -1)).astype(np.complex128)
    sx, sy = oracle.signed_freq_index(grid.nx), oracle.signed_freq_index(grid.ny)
    spec *= np.where((sy[:, None] + sx[None, :]) % 2 == 0, 1.0, -1.0) / (grid.nx * grid.ny * grid.px * grid.py)
    ref = oracle.param_grads_from_spectrum_grad(scene, grid, spec)
    out = {k: (to_numpy(got[k]), np.asarray(r)) for k, r in ref.items() if got.get(k) is not None}
    assert len(out) >= (9 if depth else 8)
    return out


@pytest.mark.parametrize("scale", [1e-20, 1e-30, 1e-36, 1e-40])
def test_smallest_field_gradients(ctx, scale):
    """Below 2^-126 FP32 numbers are steps of 2^-149.  The sums over wavelengths round products of the field
    gradient's spectrum (scale sqrt(N)) and the record's amplitude; results round once."""
    grid = Grid(1024, 1000, 8e-6, 8e-6, LAMBDAS[:1])
    scene = gwsgen.make_scene(24, grid, 51, depth_range=(-10e-3, 10e-3))
    G = (gwsgen.make_target(grid, 4242) * np.float32(scale)).astype(np.complex64)
    half = 2.0 ** -150
    det = scene.cov_xx.astype(np.float64) * scene.cov_yy - scene.cov_xy.astype(np.float64) ** 2
    amp = np.median(scene.amplitude[0] * scene.opacity * 2 * math.pi * np.sqrt(det)) / (grid.px * grid.py * grid.nx * grid.ny)
    spec = scale * math.sqrt(grid.nx * grid.ny)
    for k, (got, ref) in gradients(ctx, scene, grid, G).items():
        tol = TOL + half * math.sqrt(ref.size) / np.linalg.norm(ref)
        if k != "amplitude":
            tol += 3 * 4 * half / (spec * amp)  # a third, as above
        e = rel_l2(got, ref)
        print("  %g %s %.2e (%.2e)" % (scale, k, e, tol), flush=True)
        assert e < tol, (k, e, tol)


@pytest.mark.parametrize("ratio", [1e-3, 1e-5, 1e-6, 1e-8, 1e-12])
@pytest.mark.parametrize("depth", [True, False])
def test_wavelengths_of_different_strength(ctx, ratio, depth):
    """Each wavelength's field gradient is a gradient of its own: the same bound for the amplitudes of
    each, and, where the strong wavelengths' amplitudes vanish, for everything else."""
    grid = Grid(1024, 1000, 8e-6, 8e-6, LAMBDAS[:3])
    scene = gwsgen.make_scene(24, grid, 52, depth_range=(-10e-3, 10e-3))
    scene.amplitude[:2] = 0.0
    G = gwsgen.make_target(grid, 4243)
    G[0] *= np.float32(math.sqrt(ratio))
    G[2] *= np.float32(ratio)
    worst = {}
    for k, (got, ref) in gradients(ctx, scene, grid, G, depth).items():
        if k == "amplitude":
            for c in range(3):
                worst["amplitude[%d]" % c] = rel_l2(got[c], ref[c])
        else:
            worst[k] = rel_l2(got, ref)
    print("  %g: %s" % (ratio, {k: "%.1e" % v for k, v in worst.items()}), flush=True)
    assert max(worst.values()) < TOL, worst


def plane(grid, kx, ky):
    """exp(j 2 pi (kx x / W + ky y / H)) on the pixels, x measured from the centre pixel."""
    x, y = np.arange(grid.nx) - grid.nx // 2, np.arange(grid.ny) - grid.ny // 2
    return np.exp(2j * math.pi * ky * y / grid.ny)[:, None] * np.exp(2j * math.pi * kx * x / grid.nx)[None, :]


@pytest.mark.parametrize("waves", [[(0, 0, 1)], [(0, 0, 10)], [(0, 0, 100)], [(3, 0, 10), (-3, 0, 10)], [(0, 5, 10), (0, -5, 10)],
                                   [(0, 0, 10), (1, 0, 5), (-1, 0, 5), (0, 1, 5), (0, -1, 5)], [(-40, 0, 10), (0, 70, 10)]])
def test_mean_and_gratings(ctx, waves):
    """Field gradients of unit spread with plane waves of the given amplitudes: the waves on an axis add
    nothing to that axis' moments, so those keep the accuracy of the rest."""
    grid = Grid(1920, 1080, 8e-6, 8e-6, LAMBDAS[:1])
    sigma = (20.0, 20.0) if len(waves) == 1 else (2.0, 20.0)
    scene = gwsgen.make_scene(16, grid, 53, depth_range=(-10e-3, 10e-3), sigma_px=sigma)
    G = gwsgen.make_target(grid, 4244).astype(np.complex128)
    for kx, ky, a in waves:
        G += a * plane(grid, kx, ky)
    worst = {k: rel_l2(got, ref) for k, (got, ref) in gradients(ctx, scene, grid, G).items()}
    print("  %s: %s" % (waves, {k: "%.1e" % v for k, v in worst.items()}), flush=True)
    assert max(worst.values()) < TOL, worst


def test_largest_batch_equals_one_call_per_scene(ctx):
    """64 scenes, the most one call takes: the whole scene table."""
    import torch
    grid = Grid(1024, 1000, 8e-6, 8e-6, LAMBDAS[:1])
    scenes = [gwsgen.make_scene(1 + i % 4, grid, 700 + i) for i in range(64)]
    offsets = np.concatenate([[0], np.cumsum([s.n for s in scenes])]).tolist()
    gen = torch.Generator(device="cuda").manual_seed(1)
    G = torch.randn((64, 1, grid.ny, grid.nx), dtype=torch.complex64, device="cuda", generator=gen)
    batch = ctx.backward_batched(problem(grid), scene_to_torch(gwsgen.Scene.concat(scenes)), offsets, G)
    for s in (0, 1, 30, 62, 63):
        one = ctx.backward(problem(grid), scene_to_torch(scenes[s]), G[s].contiguous())
        for k, v in one.items():
            assert torch.equal(v, batch[k][..., offsets[s]:offsets[s + 1]]), (s, k)
