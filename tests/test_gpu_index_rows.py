"""Index of a level with more than 2^30 vertex rows, which at four threads a row is
more than one launch holds.  The mask is a full 4^4 volume, so a vertex is active
where it is a corner of a cell that holds one of 4 voxel positions along every axis
(cells are closed: a position on a vertex lies in the cells of both sides)."""
from fractions import Fraction

import pytest
import torch

pytestmark = pytest.mark.gpu


def _active(R, S):
    out = set()
    for i in range(S):
        u = Fraction(i * (R - 1), S - 1)
        for c in range(R - 1):
            if c <= u <= c + 1:
                out |= {c, c + 1}
    a = torch.zeros(R, dtype=torch.bool)
    a[sorted(out)] = True
    return a


def test_more_rows_than_a_launch_holds():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    res = [2, 1024, 1024, 1025]
    y, z, t = (_active(r, 4) for r in res[1:])
    rows = len(y) * len(z) * len(t)
    assert 1 << 30 < rows < 1 << 31 and t[-1] and z[-1] and y[-1]
    bits = torch.full((4 * 4 * 4,), 0xf, dtype=torch.int64, device="cuda")
    _idx, counts, dirs, _ = fl.fhash_build_index(fl.grid_desc([res], 1), bits, [4, 4, 4, 4])
    assert counts == [2 * int(y.sum()) * int(z.sum()) * int(t.sum())]
    zy = (z[:, None] & y[None]).flatten().long().cuda()  # rows of one active t
    before = torch.cumsum(zy, 0) - zy
    ent = dirs.view(torch.int64).view(len(t), len(zy), 2)  # one word per row: row order
    done = 0
    for k in range(len(t)):
        on = int(t[k])
        assert torch.equal(ent[k, :, 0], 3 * on * zy)
        assert torch.equal(ent[k, :, 1], 2 * (done + on * before))
        done += on * int(zy.sum())
    del _idx, dirs, ent
    torch.cuda.empty_cache()
