"""Coreset selection at the edges of its passes, bit for bit against the numpy
oracle: dilation radii either side of the two-pass limit, frames thinner than
the radius and not a multiple of the slices walked together, rows of more words
than a workgroup has threads, the last partial word, full and empty words in
the id list."""
import numpy as np
import pytest
import torch

from oracle import coreset as OC
from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


def _bits(m):
    return torch.from_numpy(synth.pack_mask_rows(m).view(np.int64)).cuda()


@pytest.mark.parametrize("shape", [(2, 2, 3, 70), (3, 9, 6, 130), (2, 17, 4, 65),
                                   (2, 8, 1100, 33)])
@pytest.mark.parametrize("r", [1, 2, 8, 9])
def test_dilation(fl, shape, r):
    T, Sz, Sy, Sx = (max(2, s) for s in shape)
    m = (np.random.default_rng(r).random((T, Sz, Sy, Sx)) < 0.004).astype(np.uint8)
    m[-1, -1, -1, -1] = m[0, 0, 0, 0] = 1
    got = fl.fhash_dilate_mask(_bits(m), [Sx, Sy, Sz, T], r)
    want = synth.pack_mask_rows(OC.dilate(m.astype(bool), r).astype(np.uint8)).view(np.int64)
    np.testing.assert_array_equal(got.cpu().numpy().ravel(), want.ravel())


@pytest.mark.parametrize("shape", [(2, 3, 5, 16500), (3, 2, 700, 9), (2, 2, 3, 64 * 255 + 1),
                                   (2, 5, 37, 190)])
def test_boxes_and_ids(fl, shape):
    T, Sz, Sy, Sx = shape
    rng = np.random.default_rng(Sx)
    m = np.zeros(shape, np.uint8)
    m[0, Sz // 2, : Sy // 2 + 1, Sx // 3:] = 1       # full words and a partial last one
    m[-1] = rng.random(shape[1:]) < 0.001
    m[-1, -1, -1, -1] = 1
    bits, dims = _bits(m), [Sx, Sy, Sz, T]
    box = fl.fhash_feature_boxes(bits, dims).cpu().numpy()
    for k in list(range(T)) + [None]:
        z, y, x = np.nonzero(m[k] if k is not None else m.any(0))
        want = ([x.min(), y.min(), z.min(), x.max(), y.max(), z.max()] if x.size
                else [Sx, Sy, Sz, -1, -1, -1])
        assert box[T if k is None else k].tolist() == want
    ids = fl.fhash_coreset(bits, dims).cpu().numpy()
    np.testing.assert_array_equal(ids, np.flatnonzero(m))
    sub = fl.fhash_coreset_frames(bits, dims, [T - 1]).cpu().numpy()
    np.testing.assert_array_equal(sub, np.flatnonzero(m[-1]) + (T - 1) * Sz * Sy * Sx)
