"""Marching 2^29 rays, which at eight threads a ray is more than one launch holds:
one image, a batch of two and a whole render.  Every ray starts inside a volume
that is all feature, so each has one sample at pace 1, and every sample a place of
its own."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DIMS = [16, 16, 16, 2]
# from the volume's centre along x: every ray has half the box in front of it
VIEW = np.array([7.5, 7.5, 7.5, 1, 0, 0, 0, 1, 0, 0, 0, 1, 0.4, 2.0], np.float32)


@pytest.fixture()
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GB of device memory")
    yield fl
    torch.cuda.empty_cache()


def _bits():
    return torch.full((2 * 16 * 16,), 0xffff, dtype=torch.int64, device="cuda")


def _begin(fl, W, H):
    ws = torch.empty(fl.fhash_render_state_bytes(W, H, DIMS), dtype=torch.uint8, device="cuda")
    rgba = torch.empty(H, W, 4, device="cuda")
    st = fl.fhash_render_begin(fl.view_struct(VIEW), 0.5, W, H, _bits(), DIMS, ws, rgba)
    assert st.n_alive == W * H
    return st, ws, rgba


def _offsets(ws, n):
    """Sample counts and first samples of the rays (16 words each: ..., off, cnt)."""
    rays = ws[:64 * n].view(torch.int32).view(n, 16)
    return rays[:, 15], rays[:, 14]


def test_one_image(fl):
    W, H = 1 << 15, 1 << 14
    st, ws, _rgba = _begin(fl, W, H)
    pos = torch.full((W * H, 4), -1.0, device="cuda")
    assert fl.fhash_render_march(st, fl.render_opts(), 1, pos, W * H) == W * H
    cnt, off = _offsets(ws, W * H)
    assert (cnt == 1).all()
    place = torch.zeros(W * H, dtype=torch.uint8, device="cuda")
    place[off.long()] = 1
    assert place.all()
    assert (pos >= 0).all() and (pos <= 1).all()


def test_batch_of_two(fl):
    W, H = 1 << 14, 1 << 14
    a, b = _begin(fl, W, H), _begin(fl, W, H)
    n = 2 * W * H
    pos = torch.full((n, 4), -1.0, device="cuda")
    counts = torch.empty(1 + fl.RENDER_BATCH_MAX, dtype=torch.int32, device="cuda")
    got = fl.fhash_render_march_batch([a[0], b[0]], [1, 1], fl.render_opts(), pos, 0, n, counts)
    assert got == [W * H, W * H]
    place = torch.zeros(n, dtype=torch.uint8, device="cuda")
    for _st, ws, _rgba in (a, b):
        cnt, off = _offsets(ws, W * H)
        assert (cnt == 1).all()
        place[off.long()] = 1
    assert place.all()
    assert (pos >= 0).all() and (pos <= 1).all()


def test_whole_render(fl):
    W, H = 1 << 15, 1 << 14
    idx, counts = fl.fhash_dense_index(fl.grid_desc([[2, 2, 2, 2]], 1))
    mlp = fl.mlp_desc([1, 32, 1])
    table = torch.zeros(sum(counts), device="cuda")
    params = torch.zeros(32 + 32 + 32 + 1, device="cuda")
    tf = torch.ones(256, 4, device="cuda")  # the first sample is opaque
    rgba = torch.empty(H, W, 4, device="cuda")
    stats, _ws = fl.fhash_render(idx, mlp, table, params, _bits(), DIMS, fl.view_struct(VIEW), 0.5,
                                 tf, W, H, fl.render_opts(), rgba)
    assert stats.samples == W * H and stats.iterations == 1
    assert (rgba == 1).all()
