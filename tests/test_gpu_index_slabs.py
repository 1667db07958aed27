"""Index build of levels much coarser than the volume, which takes the mask a slab of
frames at a time: bit for bit the directory that the same levels get beside a level of
the volume's own resolution, whose build has the whole mask in its workspace.  Levels
of 2 to as many times as there are frames."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _ws_bytes(fl, grid, dims):
    m, nb = fl.MaskDesc(), C.c_size_t(0)
    m.bits = 1 << 20
    for d in range(4):
        m.dims[d] = dims[d]
    assert fl.lib().fhash_build_index(C.byref(grid), C.byref(m), None, None, C.byref(nb), None,
                                      None, None) == fl.OK
    return nb.value


@pytest.mark.parametrize("T,res", [
    (60, [[9, 13, 5, 2], [30, 40, 11, 5], [60, 100, 30, 11], [61, 99, 31, 40]]),
    (61, [[50, 60, 20, 61], [100, 150, 25, 60], [64, 33, 9, 3]]),
    (60, [[17, 200, 60, 2]]),
])
@pytest.mark.parametrize("layout", ["rows", "bricks"])
def test_slabs_equal_whole(T, res, layout):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    dims = [480, 720, 120, T]
    words = T * 120 * 720 * 8
    lay = fl.LAYOUT_BRICKS if layout == "bricks" else fl.LAYOUT_ROWS
    coarse, both = (fl.grid_desc(r, 1, lay) for r in (res, res + [dims]))
    whole = lambda r: 8 * (words + max(T * 120 * 8 * v[1] for v in r)  # noqa: E731
                           + max(T * v[2] * 8 * v[1] for v in r))
    assert _ws_bytes(fl, coarse, dims) < whole(res)
    assert _ws_bytes(fl, both, dims) >= whole(res + [dims])
    bits = torch.zeros(words, dtype=torch.int64, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(T)
    at = torch.randint(0, words, (400,), device="cuda", generator=gen)
    bits[at] = 1 << torch.randint(0, 32, (400,), device="cuda", generator=gen)
    bits[0], bits[-1] = 1, 1 << 31  # the corners of the volume
    i0, n0, d0, _ = fl.fhash_build_index(coarse, bits, dims)
    i1, n1, d1, _ = fl.fhash_build_index(both, bits, dims)
    assert n0 == n1[:len(res)] and min(n0) > 0
    end = int(i0.dir_offset[len(res)])
    assert end == int(i1.dir_offset[len(res)])
    assert torch.equal(d0.view(-1, 2)[:end], d1.view(-1, 2)[:end])
    np.testing.assert_array_equal(list(i0.slot_offset)[:len(res) + 1],
                                  list(i1.slot_offset)[:len(res) + 1])
