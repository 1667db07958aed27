"""Claim flags of the deferred Adam set in one call, whose launch on bricks has fewer
grid rows than levels from 57,345 samples on (by the flags' number too), against the
same batch in calls of 5,000, which have a grid row per level: the same bytes."""
import numpy as np
import pytest
import torch

from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [57344, 57345, 98305, 163841])
@pytest.mark.parametrize("kind", ["rows", "bricks", "large bricks"])
def test_flags(kind, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    F = 2
    if kind == "large bricks":  # 8.7 MB of flags
        dims = [130, 128, 128, 33]
        m = np.ones(dims[::-1], np.uint8)
    else:
        dims = [70, 40, 30, 6]
        m = (np.random.default_rng(2).random(dims[::-1]) < 0.002).astype(np.uint8)
    res = [[3 + k, 3 + k, 3 + k, 2 + k // 2] for k in range(8)] + [[33, 20, 17, 4], dims]
    bits = torch.from_numpy(synth.pack_mask_rows(m).view(np.int64)).cuda()
    lay = fl.LAYOUT_ROWS if kind == "rows" else fl.LAYOUT_BRICKS
    idx, _, _keep, _ = fl.fhash_build_index(fl.grid_desc(res, F, lay), bits, dims)
    begin = int(idx.slot_offset[1]) * F // 16 * 16
    end = int(idx.slot_offset[len(res)]) * F // 16 * 16
    arrays = [torch.zeros(64, device="cuda") for _ in range(4)]  # the mark touches none
    pos = torch.rand(n, 4, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    ws = []
    for step in (n, 5000):
        lz = fl.LazyState(begin, end, 16)
        for i in range(0, n, step):
            part = pos[i:i + step]
            fl.fhash_lazy_prepare(idx, part, len(part), lz, *arrays, phases=fl.LAZY_MARK)
        ws.append(lz.ws.clone())
    clean = fl.LazyState(begin, end, 16).ws
    assert torch.equal(ws[0], ws[1])
    assert (ws[0] != clean).sum() > min((end - begin) // 64, n)
