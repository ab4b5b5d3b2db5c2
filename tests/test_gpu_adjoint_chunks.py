"""GPU parity of the adjoints with the FP64 oracle gradient where the number of Gaussians per item
changes: counts around the chunk sizes and their steps on few, more and many tiles, partial
chunks, and scenes of different chunk sizes in one batch."""
import numpy as np
import pytest

import gwsgen
import oracle
from gwsgen import Grid
from gpu_util import problem, rel_l2, scene_to_torch, to_numpy

pytestmark = pytest.mark.gpu

# as for every gradient of this size: phase roundings of 1.5e-6 per term, sums that may cancel to
# about a third of their terms' norm
TOL = 5e-6


@pytest.mark.parametrize("nx,ny,c,n,depth", [(128, 96, 2, 15, True), (256, 256, 1, 17, False),
                                             (160, 120, 3, 64, True), (256, 192, 1, 1025, True), (250, 240, 4, 130, False),
                                             (480, 360, 1, 513, False), (640, 450, 1, 257, True), (1200, 900, 1, 65, False),
                                             (1200, 900, 1, 769, True), (2000, 1600, 1, 257, True)])
def test_counts(nx, ny, c, n, depth):
    import torch
    import paper_2505_06582_amd as gws
    ctx = gws.context(0)
    grid = Grid(nx, ny, 8e-6, 8e-6, (638e-9, 520e-9, 450e-9, 570e-9)[:c])
    # the oracle sums every frequency: of twenty Gaussians, of which the scene holds copies
    few = gwsgen.make_scene(20, grid, 900 + n, depth_range=(-10e-3, 10e-3))
    src = np.arange(n) % 20
    scene = few.subset(src)
    G = gwsgen.make_target(grid, 4242)
    got = ctx.backward(problem(grid), scene_to_torch(scene), torch.from_numpy(G).cuda(), want_depth=depth)
    ref = oracle.backward(few, grid, G.astype(np.complex128))
    for k, r in ref.items():
        if got.get(k) is not None:
            e = rel_l2(to_numpy(got[k]), np.asarray(r)[..., src])
            print("  %s %.1e" % (k, e), flush=True)
            assert e < TOL, (k, e)


@pytest.mark.parametrize("nx,ny", [(256, 256), (1280, 800)])
def test_batch_of_mixed_sizes_same_bits(nx, ny):
    import torch
    import paper_2505_06582_amd as gws
    ctx = gws.context(0)
    grid = Grid(nx, ny, 8e-6, 8e-6, (520e-9,))
    counts = [5, 0, 300, 2500]
    scenes = [gwsgen.make_scene(n, grid, 70 + n) for n in counts]
    offsets = np.concatenate([[0], np.cumsum(counts)]).tolist()
    G = torch.from_numpy(np.stack([gwsgen.make_target(grid, 5 + i) for i in range(4)])).cuda()
    got = ctx.backward_batched(problem(grid), scene_to_torch(gwsgen.Scene.concat(scenes)), offsets, G)
    for i, s in enumerate(scenes):
        if counts[i] == 0:
            continue
        one = ctx.backward(problem(grid), scene_to_torch(s), G[i].contiguous())
        for k, v in one.items():
            if v is not None:
                assert torch.equal(v, got[k][..., offsets[i]:offsets[i + 1]]), (i, k)
