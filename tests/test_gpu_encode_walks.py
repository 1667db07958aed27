"""The separate encoding at the batch sizes where its launch walks samples and levels
another way (4,096, 40,960, 81,920 and 524,288 samples; groups of 65,536, in the
backward of 32,768 too): forward bit for bit, and backward with positive terms only,
against the same batch in calls of 999 samples."""
import numpy as np
import pytest
import torch

from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu

DIMS = [70, 40, 30, 6]
RES = [[3, 3, 3, 2], [9, 8, 7, 3], [33, 20, 17, 4], [70, 40, 30, 6]]


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


def _index(fl, kind, F):
    if kind == "hash":
        return fl.fhash_hash_index(fl.grid_desc(RES, F), 12)[0], None
    if kind == "large hash":  # its levels do not fit one L2 together
        return fl.fhash_hash_index(fl.grid_desc([[40, 40, 40, 40]] * 4, F), 20)[0], None
    if kind == "large dense":  # past the L2s, in four levels
        return fl.fhash_dense_index(fl.grid_desc([[60, 50, 40, 10]] * 4, F))[0], None
    m = (np.random.default_rng(2).random(DIMS[::-1]) < 0.002).astype(np.uint8)
    bits = torch.from_numpy(synth.pack_mask_rows(m).view(np.int64)).cuda()
    lay = fl.LAYOUT_BRICKS if kind == "bricks" else fl.LAYOUT_ROWS
    idx, _, dirs, _ = fl.fhash_build_index(fl.grid_desc(RES, F, lay), bits, DIMS)
    return idx, dirs


@pytest.mark.parametrize("n", [1, 257, 4096, 4097, 32769, 40960, 40961, 65537, 81921, 131073,
                               524289])
@pytest.mark.parametrize("F", [1, 2, 4, 8])
@pytest.mark.parametrize("kind", ["active", "large dense", "hash", "large hash", "bricks"])
def test_every_walk_gives_the_same(fl, kind, F, n):
    idx, _keep = _index(fl, kind, F)
    L = len(RES)
    rows = int(idx.slot_offset[L])
    gen = torch.Generator(device="cuda").manual_seed(n + F)
    pos = torch.rand(n, 4, device="cuda", generator=gen)
    table = torch.rand(rows * F, device="cuda", generator=gen) - 0.5
    got = torch.full((n, L * F), 9.0, device="cuda")
    want = torch.empty_like(got)
    grad = 1.0 + torch.rand(n, L * F, device="cuda", generator=gen)
    dgot, dwant = (torch.zeros(rows * F, device="cuda") for _ in range(2))
    fl.fhash_encode_fwd(idx, pos, n, table, got)
    fl.fhash_encode_bwd(idx, pos, n, grad, dgot)
    for i in range(0, n, 999):
        k = min(999, n - i)
        part = torch.empty(k, L * F, device="cuda")
        fl.fhash_encode_fwd(idx, pos[i:i + k], k, table, part)
        want[i:i + k] = part
        fl.fhash_encode_bwd(idx, pos[i:i + k], k, grad[i:i + k].contiguous(), dwant)
    assert torch.equal(got, want)
    # positive terms: the sums of the n L 16 F products in any order lie within
    # (terms of a vertex) 2^-24 of themselves; 524,289 samples on the 54 vertices of
    # the coarsest level reach 4e5 terms, whose rounding errors add up at random:
    # 6e-8 sqrt(4e5) = 4e-5
    assert torch.allclose(dgot, dwant, rtol=1e-4, atol=0)
