"""Dilation on both sides of the rule that gives the z direction a pass of its own
(slices that fit the LDS copy and slices that do not, frames of one and of several
groups of 8 slices), bit for bit against a three-dimensional maximum filter."""
import numpy as np
import pytest
import torch

from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 3, 5, 8, 9])
@pytest.mark.parametrize("dims", [
    (40, 30, 20, 4),      # one pass below r = 8
    (200, 200, 20, 3),    # the two cross between
    (64, 2000, 9, 2),     # two passes from r = 1
    (70, 4100, 7, 2),     # past the LDS copy: two passes always
    (65, 3000, 2, 2),     # frames thinner than the radius
])
def test_against_maximum_filter(dims, r):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    Sx, Sy, Sz, T = dims
    m = (np.random.default_rng(r + Sy).random((T, Sz, Sy, Sx)) < 0.1 / (2 * r + 1) ** 3)
    m[0, 0, 0, 0] = m[-1, -1, -1, -1] = True
    got = fl.fhash_dilate_mask(
        torch.from_numpy(synth.pack_mask_rows(m.astype(np.uint8)).view(np.int64)).cuda(),
        list(dims), r)
    want = torch.from_numpy(m.astype(np.float32))[:, None]
    for d in range(3):  # the cube is separable
        k, p = [1, 1, 1], [0, 0, 0]
        k[d], p[d] = 2 * r + 1, r
        want = torch.nn.functional.max_pool3d(want, k, 1, p)
    want = synth.pack_mask_rows(want[:, 0].numpy().astype(np.uint8)).view(np.int64)
    np.testing.assert_array_equal(got.cpu().numpy().ravel(), want.ravel())
