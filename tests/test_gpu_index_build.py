"""The index build at the edges of its passes, against the oracle's active set
vertex by vertex: rows of more words than a transposition tile, vertices whose
voxel range spans several words, one vertex per voxel, levels finer than the
volume, rows that do not fill a workgroup, a single level, both slot orders."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


VOLUMES = {
    "wide": ((2100, 70, 3, 2), [[2, 2, 2, 2], [5, 70, 3, 2], [700, 9, 2, 2], [2100, 70, 3, 2]]),
    "finer": ((130, 5, 4, 3), [[64, 5, 4, 3], [129, 3, 2, 2], [130, 5, 4, 3], [300, 11, 6, 5]]),
    "one level": ((64, 65, 2, 2), [[64, 65, 2, 2]]),
    "many levels": ((97, 66, 9, 5), [[3 + 4 * k, 2 + 3 * k, 2 + k // 3, 2 + k // 6]
                                     for k in range(20)]),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("name", VOLUMES)
@pytest.mark.parametrize("density", [0.0008, 0.2])
def test_directory_holds_the_oracles_active_set(fl, name, density, layout):
    (Sx, Sy, Sz, T), res = VOLUMES[name]
    rng = np.random.default_rng(len(name))
    mask = (rng.random((T, Sz, Sy, Sx)) < density).astype(np.uint8)
    mask[-1, -1, -1, -1] = 1
    bits = torch.from_numpy(synth.pack_mask_rows(mask).view(np.int64)).cuda()
    grid = fl.grid_desc(res, 2, layout)
    idx, counts, dirs, _ = fl.fhash_build_index(grid, bits, [Sx, Sy, Sz, T])
    words = dirs.cpu().numpy().view(np.uint64)
    for l, (rx, ry, rz, rt) in enumerate(res):
        want, n = O.level_slots(res[l], mask, layout)
        assert counts[l] == n
        t, z, y, x = np.meshgrid(*(np.arange(r) for r in (rt, rz, ry, rx)), indexing="ij")
        if layout == 0:
            wv = (rx + 63) // 64
            at, bit = ((t * rz + z) * wv + x // 64) * ry + y, x % 64
        else:
            by, bz = (ry + 1) // 2, (rz + 1) // 2
            wb = ((rx + 1) // 2 + 3) // 4
            at = (((t // 2) * bz + z // 2) * wb + x // 8) * by + y // 2
            bit = 16 * (x // 2 % 4) + x % 2 + 2 * (y % 2) + 4 * (z % 2) + 8 * (t % 2)
        ent = words[int(idx.dir_offset[l]) + at.ravel()]
        b = bit.ravel().astype(np.uint64)
        below = ent[:, 0] & ((np.uint64(1) << b) - np.uint64(1))
        pop = np.unpackbits(below.view(np.uint8).reshape(-1, 8), axis=1).sum(1)
        slot = np.where((ent[:, 0] >> b) & np.uint64(1), ent[:, 1].astype(np.int64) + pop, -1)
        np.testing.assert_array_equal(slot, np.asarray(want).ravel(), err_msg=f"level {l}")
