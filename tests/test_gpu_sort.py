"""Order of the Gaussians in the forward: with distinct keys the field of a shuffled scene has the
same bits, at counts around its steps of keys per thread, its change to many blocks
(12288 keys), their size (4096) and the change to a scanned table (512 blocks)."""
import numpy as np
import pytest

import gwsgen
from gwsgen import Grid
from gpu_util import problem, scene_to_torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 257, 4095, 4096, 4097, 8193, 12288, 12289, 50000, 512 * 4096, 512 * 4096 + 1])
def test_shuffled_input_same_bits(n):
    import torch
    import paper_2505_06582_amd as gws
    ctx = gws.context(0)
    grid = Grid(64, 48, 8e-6, 8e-6, (520e-9,))
    scene = gwsgen.make_scene(n, grid, 11)
    rng = np.random.default_rng(n)
    # distinct depths of both signs: exact multiples of 2^-28 m
    scene.depth[:] = ((rng.permutation(n) - n // 2) * 2.0 ** -28).astype(np.float32)
    g = scene_to_torch(scene)
    p = torch.from_numpy(rng.permutation(n)).cuda()
    shuffled = {k: v[..., p].contiguous() for k, v in g.items()}
    a, b = ctx.forward(problem(grid), g), ctx.forward(problem(grid), shuffled)
    assert torch.isfinite(torch.view_as_real(a)).all() and float(a.abs().max()) > 0
    assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
