"""GPU parity of the matrix-core adjoint with the FP64 oracle gradient at the sizes where it can go
wrong: chunks around 512 Gaussians, passes of 16, each class of the cross term, ragged grids, deep
Gaussians, zero amplitudes, every number of wavelengths, with and without the depth gradient."""
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


def check(ctx, scene, grid, label, depth, **kw):
    import torch
    G = gwsgen.make_target(grid, 4242)
    got = ctx.backward(problem(grid, **kw), scene_to_torch(scene), torch.from_numpy(G).cuda(), want_depth=depth)
    ref = oracle.backward(scene, grid, G.astype(np.complex128))
    worst = {}
    for k, r in ref.items():
        if got.get(k) is not None:
            worst[k] = rel_l2(to_numpy(got[k]), r)
    print("  %s: %s" % (label, {k: "%.1e" % v for k, v in worst.items()}), flush=True)
    assert len(worst) >= 8 and max(worst.values()) < TOL, (label, worst)


@pytest.mark.parametrize("nx,ny,c,n,depth", [(1024, 1000, 1, 1, True), (1200, 900, 2, 15, True), (1024, 1000, 3, 17, True),
                                             (1440, 720, 4, 33, False), (1024, 1000, 1, 257, False),
                                             (1000, 1024, 1, 513, True), (1152, 960, 2, 40, False)])
def test_counts_and_ragged_grids(ctx, nx, ny, c, n, depth):
    grid = Grid(nx, ny, 8e-6, 8e-6, LAMBDAS[:c])
    scene = gwsgen.make_scene(n, grid, 500 + n, depth_range=(-10e-3, 10e-3))
    check(ctx, scene, grid, "%dx%dx%d n=%d" % (nx, ny, c, n), depth)


@pytest.mark.parametrize("a", [0.0, 0.0174, 0.0176, 0.0799, 0.0801, 0.1201, 0.2001, 0.3499, 0.3501])
def test_cross_term_classes(ctx, a):
    """Both signs of exp(-a t) on a 16 x 16 sub-tile, |t| <= 1, among Gaussians without a cross term."""
    grid = Grid(1280, 1024, 8e-6, 8e-6, (520e-9,))
    scene = gwsgen.make_scene(40, grid, 78, depth_range=(-8e-3, 8e-3), sigma_px=(4.0, 4.0))
    sxy = a * grid.nx * grid.px * grid.ny * grid.py / (56.25 * 4 * math.pi ** 2)
    scene.cov_xx[:20] = scene.cov_yy[:20] = np.float32(1.3 * sxy + (4.0 * grid.px) ** 2)
    scene.cov_xy[:20] = np.float32(sxy) * np.where(np.arange(20) % 2 == 0, 1, -1)
    check(ctx, scene, grid, "a=%g" % a, True)


def test_deep_zero_amplitude_and_reference_wave(ctx):
    grid = Grid(1024, 1000, 8e-6, 8e-6, LAMBDAS[:2], ref_nu=(9e3, -4e3))
    scene = gwsgen.make_scene(48, grid, 10, depth_range=(-10e-3, 10e-3))
    scene.depth[::6] = np.float32(0.3)      # outside the separable form's depth
    scene.amplitude[:, 1::5] = 0.0          # their amplitude gradients do not vanish
    scene.opacity[2::7] = 0.0
    check(ctx, scene, grid, "deep, zero amplitudes, reference wave", True)


def test_repeats_bitwise_and_batched(ctx):
    import torch
    grid = Grid(1024, 1000, 8e-6, 8e-6, LAMBDAS[:2])
    counts = [1500, 0, 41]
    scenes = [gwsgen.make_scene(n, grid, 90 + n) for n in counts]
    G = torch.from_numpy(np.stack([gwsgen.make_target(grid, 7 + s) for s in range(3)])).cuda()
    g = scene_to_torch(gwsgen.Scene.concat(scenes))
    batch = ctx.backward_batched(problem(grid), g, [0, 1500, 1500, 1541], G)
    for s, (lo, hi) in enumerate(((0, 1500), (1500, 1500), (1500, 1541))):
        if hi > lo:
            for _ in range(2):
                one = ctx.backward(problem(grid), scene_to_torch(scenes[s]), G[s].contiguous())
                for k, v in one.items():
                    assert torch.equal(v, batch[k][..., lo:hi]), (s, k)
