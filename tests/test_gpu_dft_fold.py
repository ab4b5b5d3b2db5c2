"""The split-bf16 DFT's radix step and folding at the lengths where they change form: N / R even (a
term that is its own mirror) and odd, R = 4 and R = 2, halves around the block tile's 64 frequencies
and 32 terms, one and several images, in place."""
import numpy as np
import pytest

from gpu_util import rel_l2, to_numpy

pytestmark = pytest.mark.gpu

# hi lo splits leave 2^-17 of each operand (uniform: / sqrt(3)) and drop lo lo, in two products and two
# axes; the sums' roundings are far below
TOL = 4 * 2.0 ** -17


@pytest.mark.parametrize("ny,nx,batch", [(16, 20, 3), (18, 36, 1), (30, 60, 2), (120, 128, 1), (250, 480, 1), (256, 500, 1),
                                         (60, 486, 1), (500, 512, 2), (90, 1024, 1), (540, 54, 2)])
@pytest.mark.parametrize("direction", [1, -1])
def test_lengths(ny, nx, batch, direction):
    import torch
    import paper_2505_06582_amd as gws
    ctx = gws.context(0)
    rng = np.random.default_rng(ny * nx + direction)
    x = (rng.standard_normal((batch, ny, nx)) + 1j * rng.standard_normal((batch, ny, nx))).astype(np.complex64)
    ref = np.fft.ifft2(x.astype(np.complex128)) * (nx * ny) if direction > 0 else np.fft.fft2(x.astype(np.complex128))
    t = torch.from_numpy(x).cuda()
    got = ctx.dft2d(t, direction, xform=gws.XFORM_DFT_BF16X3)
    assert rel_l2(to_numpy(got), ref) < TOL
    ctx.dft2d(t, direction, xform=gws.XFORM_DFT_BF16X3, out=t)
    assert torch.equal(torch.view_as_real(t), torch.view_as_real(got))
