"""GPU parity of the matrix-core spectrum accumulation with the FP64 oracle where the scales of its
factors can go wrong: supports of a few frequencies (an envelope that falls by many powers of two within
a sub-tile), record amplitudes down to FP32's smallest numbers, wavelengths of very different
strength, sub-tiles whose centre lies beyond the grid."""
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


def spectra(ctx, scene, grid, mx, my):
    """(the library's spectrum at centred indices, the oracle's), and the field must be finite."""
    import torch
    mx, my = (mx % grid.nx).astype(np.int32), (my % grid.ny).astype(np.int32)
    field, spec = ctx.forward(problem(grid), scene_to_torch(scene), want_spectrum=True)
    assert bool(torch.isfinite(torch.view_as_real(field)).all())
    return to_numpy(spec)[:, my, mx], oracle_dft_ready(scene, grid, mx, my)


def block(half):
    m = np.arange(-half, half + 1)
    my, mx = np.meshgrid(m, m, indexing="ij")
    return mx.ravel(), my.ravel()


def wide(grid, frac, seed):
    """One Gaussian of standard deviation frac * W on both axes."""
    g = gwsgen.make_scene(1, grid, seed, depth_range=(-5e-3, 5e-3))
    g.cov_xx[:] = g.cov_yy[:] = np.float32((frac * grid.nx * grid.px) ** 2)
    g.cov_xy[:] = 0.0
    g.amplitude[:] = 0.5
    g.opacity[:] = 1.0
    return g


@pytest.mark.parametrize("frac", [0.1, 0.15, 0.2, 0.25, 0.3, 0.5])
def test_one_wide_gaussian(ctx, frac):
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:2])
    got, ref = spectra(ctx, wide(grid, frac, 4), grid, *block(20))
    assert rel_l2(got, ref) < TOL


@pytest.mark.parametrize("n", [2, 129, 1025])
def test_a_wide_gaussian_after_ordinary_ones(ctx, n):
    """The widest is last in the order: alone in its tile's last chunk of 128 for 129 and 1025."""
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:1])
    scene = gwsgen.Scene.concat([gwsgen.make_scene(n - 1, grid, 40 + n, sigma_px=(17.0, 20.0)), wide(grid, 0.2, 5)])
    got, ref = spectra(ctx, scene, grid, *block(20))
    assert rel_l2(got, ref) < TOL


def test_faint_ordinary_gaussians_under_a_wide_one(ctx):
    """Where the wide one's support ends (8 to 40 frequencies from DC) only the ordinary ones are left:
    the scale there must be the wide one's value there, not its peak."""
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:1])
    scene = gwsgen.Scene.concat([gwsgen.make_scene(60, grid, 6), wide(grid, 0.2, 5)])
    scene.amplitude[:, :60] *= np.float32(1e-3)
    mx, my = block(40)
    far = np.hypot(mx, my) > 8
    got, ref = spectra(ctx, scene, grid, mx[far], my[far])
    assert rel_l2(got, ref) < TOL


@pytest.mark.parametrize("log2amp", [-100, -118, -122, -124, -126, -128, -130, -136, -140])
@pytest.mark.parametrize("zero", [False, True])
def test_smallest_amplitudes(ctx, log2amp, zero):
    """Record amplitudes of 2^log2amp, alone on their sub-tiles or beside a wavelength of amplitude 0.  Record
    and spectrum are FP32 numbers, below 2^-126 in steps of 2^-149: half a step each, of values
    that are 2^-6 of the amplitude where the support's energy is."""
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:2])
    scene = gwsgen.make_scene(3, grid, 21, sigma_px=(6.0, 8.0), depth_range=(-5e-3, 5e-3))
    det = scene.cov_xx.astype(np.float64) * scene.cov_yy - scene.cov_xy.astype(np.float64) ** 2
    norm = 2 * math.pi * np.sqrt(det) / (grid.px * grid.py * grid.nx * grid.ny)
    scene.opacity[:] = 1.0
    scene.amplitude[:] = (2.0 ** log2amp / norm).astype(np.float32)
    if zero:
        scene.amplitude[1] = 0.0
    rng = np.random.default_rng(3)
    got, ref = spectra(ctx, scene, grid, rng.integers(-100, 100, 700), rng.integers(-80, 80, 700))
    step = 2.0 ** -149 / 2.0 ** log2amp
    err = rel_l2(got[0], ref[0])
    print("  2^%d: %.3e" % (log2amp, err), flush=True)
    assert err < TOL + (0.5 + 0.5 * 64) * step
    if zero:
        assert not np.any(got[1])


@pytest.mark.parametrize("log2amp", [-40, -90, -120])
def test_a_faint_wide_gaussian(ctx, log2amp):
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:1])
    scene = wide(grid, 0.25, 4)
    norm = 2 * math.pi * float(scene.cov_xx[0]) / (grid.px * grid.py * grid.nx * grid.ny)
    scene.amplitude[:] = np.float32(2.0 ** log2amp / norm)
    got, ref = spectra(ctx, scene, grid, *block(20))
    assert rel_l2(got, ref) < TOL


@pytest.mark.parametrize("ratio", [1e-2, 1e-3, 1e-4, 1e-5, 1e-6, 1e-8, 1e-20, 1e-35])
def test_wavelengths_of_different_strength(ctx, ratio):
    """Each wavelength is a sum of its own: the same bound for each."""
    grid = Grid(2400, 1800, 8e-6, 8e-6, LAMBDAS[:3])
    scene = gwsgen.make_scene(150, grid, 31, depth_range=(-10e-3, 10e-3))
    scene.amplitude[0] *= np.float32(math.sqrt(ratio))
    scene.amplitude[2] *= np.float32(ratio)
    rng = np.random.default_rng(4)
    got, ref = spectra(ctx, scene, grid, rng.integers(-300, 300, 700), rng.integers(-225, 225, 700))
    errs = [rel_l2(got[c], ref[c]) for c in range(3)]
    print("  %g: %s" % (ratio, errs), flush=True)
    # 1e-35: record amplitudes near 1e-40, in steps of 2^-149, half a step for record and result each (values
    # 2^-6 of the amplitude)
    norm = 2 * math.pi * np.sqrt(np.median(scene.cov_xx.astype(np.float64) * scene.cov_yy)) / (grid.px * grid.py * grid.nx * grid.ny)
    for c, r in ((0, math.sqrt(ratio)), (1, 1.0), (2, ratio)):
        assert errs[c] < TOL + 33 * 2.0 ** -149 / (r * 0.25 * norm), (c, errs)


@pytest.mark.parametrize("nx,ny", [(2500, 1800), (2500, 2500), (3750, 1250)])
def test_sub_tiles_beyond_the_propagating_disk(ctx, nx, ny):
    """Half sizes of 16 i + 1 ... 7: the outermost sub-tiles' centres lie beyond the grid, and with a pitch
    just above lambda / sqrt(2) beyond 1 / lambda, though every grid frequency propagates."""
    lam = 520e-9
    p = lam / math.sqrt(2.0) * 1.001
    grid = Grid(nx, ny, p, p, (lam,))
    scene = gwsgen.make_scene(40, grid, 12, depth_range=(-10e-6, 10e-6), sigma_px=(0.5, 0.8))
    rng = np.random.default_rng(5)
    hx, hy = nx // 2, ny // 2
    mx = np.concatenate([rng.integers(-hx, hx, 500), rng.integers(hx - 16, hx, 200)])
    my = np.concatenate([rng.integers(-hy, hy, 500), rng.integers(-hy, -hy + 16, 200)])
    got, ref = spectra(ctx, scene, grid, mx, my)
    # at the disk's edge k_z falls by 0.1 / lambda within a sub-tile: 2 revolutions at 10 um, as above
    assert rel_l2(got, ref) < TOL
