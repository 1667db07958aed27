"""Samples of the march ray by ray, as the rays' own first sample and count give
them: at every pace, in the single and the batched march, the runs of a ray one
after another are the same sequence as at pace 1, which goes forward along the ray
and has as many samples as the oracle renderer composites in that pixel; and the
runs of a march's rays share no sample."""
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


def _rays(ws, n):
    """(ox oy oz dx dy dz s0 s1) and (k, pixel, off, cnt) of every ray; ray r is pixel r."""
    r = ws[:64 * n].cpu().numpy().reshape(n, 64)
    return r[:, :32].copy().view(np.float32).astype(np.float64), r[:, 48:].copy().view(np.int32)


def _march(fl, bits, dims, view, t, W, H, pace, ds, max_steps, batched):
    """Every ray's samples in the order it emits them, and the rays."""
    n = W * H
    ws = torch.empty(fl.fhash_render_state_bytes(W, H, dims), dtype=torch.uint8, device="cuda")
    rgba = torch.empty(H, W, 4, device="cuda")
    st = fl.fhash_render_begin(fl.view_struct(view), t, W, H, bits, dims, ws, rgba)
    opts = fl.render_opts(ds=ds, arm_max=1000, max_steps=max_steps)
    pos = torch.empty(n * pace, 4, device="cuda")
    y = torch.zeros(n * pace, device="cuda")
    tf = torch.zeros(256, 4, device="cuda")  # nothing is opaque: rays run to their end
    counts = torch.empty(1 + fl.RENDER_BATCH_MAX, dtype=torch.int32, device="cuda")
    geo, _ = _rays(ws, n)
    alive = geo[:, 6] < geo[:, 7]
    out = [[np.zeros((0, 4), np.float32)] for _ in range(n)]
    while st.n_alive > 0:
        assert st.n_alive == alive.sum()
        if batched:
            ns = fl.fhash_render_march_batch([st], [pace], opts, pos, 0, n * pace, counts)[0]
        else:
            ns = fl.fhash_render_march(st, opts, pace, pos, n * pace)
        p, (_, state) = pos[:ns].cpu().numpy(), _rays(ws, n)
        used = np.zeros(ns, int)
        for r in np.flatnonzero(alive):
            off, cnt = state[r, 2], state[r, 3]
            ended, cnt = bool(cnt >> 30), cnt & ((1 << 30) - 1)
            assert cnt <= pace and (ended or cnt == pace)
            out[r].append(p[off:off + cnt])
            used[off:off + cnt] += 1
            alive[r] = not ended
        assert (used == 1).all()
        if batched:
            fl.fhash_render_composite_batch([st], y, [tf], opts, [rgba], counts)
        else:
            fl.fhash_render_composite(st, y, tf, opts, rgba)
    assert not alive.any()
    return [np.concatenate(o) for o in out], geo


@pytest.mark.parametrize("W,H,density,ds,max_steps", [
    (16, 8, 0.002, 0.5, 1 << 20),    # 128 rays: one workgroup
    (43, 3, 0.0, 0.05, 1 << 20),     # 129 rays; runs of hundreds of steps
    (9, 7, 0.3, 0.5, 61),            # the lattice cut inside the volume
    (5, 1, 1.0, 3.0, 1 << 20),       # fewer steps than lanes on some rays
    (3, 2, 0.004, 0.02, 1 << 20),    # runs of single steps far apart, past the kept 64
])
def test_rays_emit_their_steps_in_order(fl, W, H, density, ds, max_steps):
    mask = _mask(density)
    dims = list(mask.shape[::-1])
    bits = torch.from_numpy(synth.pack_mask_rows(mask).view(np.int64)).cuda()
    view = synth.orbit_view(dims, 0.9, 0.35, W, H)
    t = 0.75
    want, geo = _march(fl, bits, dims, view, t, W, H, 1, ds, max_steps, False)
    g = O.Grid(np.array([[2, 2, 2, 2]]), 1)
    width = [1, 16, 1]
    _, _, _, pix = O.render(g, np.zeros((16, 1)), width, np.zeros(O.mlp_num_params(width)), mask,
                            view, t, np.zeros((256, 4), np.float32), W, H, ds=ds,
                            max_steps=max_steps, pixel_stats=True)
    assert [len(w) for w in want] == [int(k) for k in pix[..., 0].ravel()]
    assert max(len(w) for w in want) > (64 if ds < 0.1 else 0)
    for w, r in zip(want, geo):  # the lattice steps of the samples: each later than the last
        p = w[:, :3].astype(np.float64) * (np.array(dims[:3]) - 1)
        k = ((p - r[:3]) @ r[3:6] - r[6]) / ds - 0.5
        assert (np.abs(k - np.rint(k)) < 0.05).all() and (np.diff(np.rint(k)) > 0).all()
    for pace in (7, 64, 65, 333):
        for batched in (False, True):
            got, _ = _march(fl, bits, dims, view, t, W, H, pace, ds, max_steps, batched)
            for a, b in zip(got, want):
                np.testing.assert_array_equal(a, b)
