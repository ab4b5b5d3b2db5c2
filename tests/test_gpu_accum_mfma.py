"""GPU parity of the matrix-core spectrum accumulation with the FP64 oracle, at the sizes where it can
go wrong: list lengths around its passes of 16 and batches of 64 Gaussians, each class of the
covariance's cross term and both sides of its limits, ragged grids, mixed amplitudes, deep and off-axis
Gaussians, every number of wavelengths."""
import math

import numpy as np
import pytest

import gwsgen
from gwsgen import Grid
from gpu_util import oracle_dft_ready, problem, rel_l2, scene_to_torch, to_numpy

pytestmark = pytest.mark.gpu

# A term's factors carry 1e-7 rms each from the polynomial and the fp16 pairs; the phase's FP32
# roundings (three at up to 4 revolutions, 2^-22 of a revolution each, 2 pi / sqrt(3)) are 1.5e-6 at
# most and half of that in the mean.  2e-6 bounds their sum.
TOL = 2e-6
LAMBDAS = (638e-9, 520e-9, 450e-9, 570e-9)


@pytest.fixture(scope="module")
def ctx():
    import torch
    import paper_2505_06582_amd as gws
    assert torch.cuda.is_available()
    return gws.context(0)


def spectrum_error(ctx, scene, grid, label, n_freq=700, half_width=None, seed=5, **kw):
    """Relative L2 of the spectrum over random frequencies (|m'| <= half_width along each axis)."""
    rng = np.random.default_rng(seed)
    hx, hy = (grid.nx // 2, grid.ny // 2) if half_width is None else half_width
    mx = (rng.integers(-hx, hx, n_freq) % grid.nx).astype(np.int32)
    my = (rng.integers(-hy, hy, n_freq) % grid.ny).astype(np.int32)
    _, spec = ctx.forward(problem(grid, **kw), scene_to_torch(scene), want_spectrum=True)
    e = rel_l2(to_numpy(spec)[:, my, mx], oracle_dft_ready(scene, grid, mx, my))
    print("  %s: spectrum rel %.3e" % (label, e), flush=True)
    return e


@pytest.mark.parametrize("nx,ny,c,n", [(2400, 1800, 1, 1), (2400, 1800, 2, 15), (3000, 1440, 3, 16), (2400, 1800, 4, 17),
                                       (2160, 1944, 3, 63), (3000, 1458, 2, 65), (2400, 1800, 1, 129), (2880, 1800, 4, 1025),
                                       (4050, 1080, 1, 2600)])
def test_list_lengths_and_ragged_grids(ctx, nx, ny, c, n):
    grid = Grid(nx, ny, 8e-6, 8e-6, LAMBDAS[:c])
    scene = gwsgen.make_scene(n, grid, 300 + n, depth_range=(-10e-3, 10e-3))
    assert spectrum_error(ctx, scene, grid, "%dx%dx%d n=%d" % (nx, ny, c, n), half_width=(nx // 8, ny // 8)) < TOL


@pytest.mark.parametrize("a", [0.0, 0.004, 0.0174, 0.0176, 0.05, 0.0799, 0.0801, 0.1199, 0.1201, 0.1999, 0.2001, 0.3499,
                               0.3501, 0.8])
@pytest.mark.parametrize("sign", [1, -1])
def test_cross_term_classes(ctx, a, sign):
    """Gaussians whose cross term on a 16 x 16 sub-tile is exactly exp(-a t), |t| <= 1."""
    grid = Grid(2560, 2048, 8e-6, 8e-6, (520e-9,))
    scene = gwsgen.make_scene(40, grid, 77, depth_range=(-8e-3, 8e-3), sigma_px=(4.0, 4.0))
    sxy = a * grid.nx * grid.px * grid.ny * grid.py / (56.25 * 4 * math.pi ** 2)
    var = 1.3 * sxy + (4.0 * grid.px) ** 2
    scene.cov_xx[:] = scene.cov_yy[:] = np.float32(var)
    scene.cov_xy[:] = np.float32(sign * sxy)
    hw = int(0.3 * grid.nx * grid.px / math.sqrt(var) / (2 * math.pi) * 6)
    assert spectrum_error(ctx, scene, grid, "a=%g" % (sign * a), half_width=(max(16, min(hw, 640)),) * 2) < TOL


def test_nearly_singular_covariance(ctx):
    """Correlation 0.99: evaluated term by term.  The exponent's terms are 1 / (1 - 0.99) times its value
    (at most 2 where the spectrum's energy is); six roundings of 2^-24 of them, the record's included."""
    grid = Grid(2560, 2048, 8e-6, 8e-6, (520e-9,))
    scene = gwsgen.make_scene(60, grid, 78, depth_range=(-8e-3, 8e-3), sigma_px=(4.0, 4.0))
    scene.cov_xx[:] = scene.cov_yy[:] = np.float32((20 * grid.px) ** 2)
    scene.cov_xy[:] = np.float32(0.99) * scene.cov_xx
    hw = int(grid.nx / (2 * math.pi * 20) * 3)
    assert spectrum_error(ctx, scene, grid, "singular", half_width=(hw, hw)) < 200 * 2.0 * math.log(2) * 6 * 2.0 ** -24


def test_mixed_amplitudes_depths_and_reference_wave(ctx):
    """Amplitudes over forty orders of magnitude in one list, Gaussians at 0.5 m (outside the separable
    form's depth) among ordinary ones, a tilted reference wave."""
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:2])
    scene = gwsgen.make_scene(200, grid, 9, depth_range=(-10e-3, 10e-3))
    assert spectrum_error(ctx, scene, Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:2], ref_nu=(9e3, -4e3)), "reference wave",
                          half_width=(120, 90)) < TOL
    scene.depth[::7] = np.float32(0.5)
    assert spectrum_error(ctx, scene, grid, "deep", half_width=(120, 90)) < 1e-5
    rng = np.random.default_rng(3)
    scene.depth[::7] = 0.0
    scene.amplitude[:] *= np.float32(10.0) ** rng.uniform(-20, 20, scene.amplitude.shape).astype(np.float32)
    assert spectrum_error(ctx, scene, grid, "amplitudes 1e-20 ... 1e20", half_width=(120, 90)) < TOL
    scene.amplitude[:, 50] = np.float32(2e35)
    assert spectrum_error(ctx, scene, grid, "amplitude 2e35", half_width=(120, 90)) < 1e-5


def test_repeats_bitwise_and_batched(ctx):
    import torch
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:2])
    counts = [3000, 0, 41]
    scenes = [gwsgen.make_scene(n, grid, 60 + n) for n in counts]
    g = scene_to_torch(gwsgen.Scene.concat(scenes))
    fields = ctx.forward_batched(problem(grid), g, [0, 3000, 3000, 3041])
    for s, scene in enumerate(scenes):
        one = ctx.forward(problem(grid), scene_to_torch(scene))
        assert torch.equal(torch.view_as_real(one), torch.view_as_real(fields[s]))
        assert torch.equal(torch.view_as_real(one), torch.view_as_real(ctx.forward(problem(grid), scene_to_torch(scene))))
