"""The march at the edges of its work split (8 lanes and steps per ray, 128 rays
per workgroup, 64 steps kept from a ray's first sample): whatever the pace, the
rays emit the occupied lattice steps, each once and in order, and as many as
the oracle renderer composites when nothing is opaque."""
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


def _mask(density):
    m = (np.random.default_rng(3).random((3, 20, 31, 70)) < density).astype(np.uint8)
    m[:, 4:9, 10:20, 5:60] = 1  # a run far longer than 64 steps, and gaps around it
    return m


def _collect(fl, bits, dims, view, t, W, H, pace, ds, max_steps, batched):
    """Samples of every ray in the order it emits them, by pixel."""
    ws = torch.empty(fl.fhash_render_state_bytes(W, H, dims), dtype=torch.uint8, device="cuda")
    rgba = torch.empty(H, W, 4, device="cuda")
    st = fl.fhash_render_begin(fl.view_struct(view), t, W, H, bits, dims, ws, rgba)
    opts = fl.render_opts(ds=ds, arm_max=1000, max_steps=max_steps)
    cap = W * H * pace
    pos = torch.full((cap, 4), float("nan"), device="cuda")
    y = torch.zeros(cap, device="cuda")
    tf = torch.zeros(256, 4, device="cuda")  # nothing is opaque: rays run to their end
    counts = torch.empty(1 + fl.RENDER_BATCH_MAX, dtype=torch.int32, device="cuda")
    out, total = [], 0
    while st.n_alive > 0:
        if batched:
            ns = fl.fhash_render_march_batch([st], [pace], opts, pos, 0, cap, counts)[0]
        else:
            ns = fl.fhash_render_march(st, opts, pace, pos, cap)
        p = pos[:ns].cpu().numpy()
        assert np.isfinite(p).all()
        out.append(p)
        total += ns
        if batched:
            fl.fhash_render_composite_batch([st], y, [tf], opts, [rgba], counts)
        else:
            fl.fhash_render_composite(st, y, tf, opts, rgba)
    p = np.concatenate(out)
    return p[np.lexsort(p.T)], total


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("W,H,density,ds,max_steps", [
    (16, 8, 0.002, 0.5, 1 << 20),    # 128 rays: one workgroup
    (43, 3, 0.0, 0.05, 1 << 20),     # 129 rays; runs of hundreds of steps
    (9, 7, 0.3, 0.5, 61),            # the lattice cut inside the volume
    (5, 1, 1.0, 3.0, 1 << 20),       # fewer steps than lanes on some rays
])
def test_every_pace_emits_the_same_samples(fl, W, H, density, ds, max_steps, batched):
    mask = _mask(density)
    dims = list(mask.shape[::-1])
    bits = torch.from_numpy(synth.pack_mask_rows(mask).view(np.int64)).cuda()
    view = synth.orbit_view(dims, 0.9, 0.35, W, H)
    t = 0.75
    want, n = _collect(fl, bits, dims, view, t, W, H, 1, ds, max_steps, False)
    for pace in (7, 64, 65, 333):
        got, k = _collect(fl, bits, dims, view, t, W, H, pace, ds, max_steps, batched)
        assert k == n
        np.testing.assert_array_equal(got, want)
    g = O.Grid(np.array([[2, 2, 2, 2]]), 1)
    width = [1, 16, 1]
    _, _, _, pix = O.render(g, np.zeros((16, 1)), width, np.zeros(O.mlp_num_params(width)), mask,
                            view, t, np.zeros((256, 4), np.float32), W, H, ds=ds,
                            max_steps=max_steps, pixel_stats=True)
    assert n == int(pix[..., 0].sum()) and n > 0
