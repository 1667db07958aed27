"""Whole renders either side of the ray count from which the host looks after the first
iteration: image and statistics are those of the step calls, with the feature in view
and with none of it."""
import numpy as np
import pytest
import torch

from paper_2507_03836_amd import synth
from test_gpu_render import scene  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(362, 362), (363, 362)])  # 2^17 = 131,072 rays between
@pytest.mark.parametrize("mask", ["feature", "empty"])
def test_whole_render_equals_steps(scene, W, H, mask):  # noqa: F811
    s, fl = scene, scene["fl"]
    bits = s["bits"] if mask == "feature" else torch.zeros_like(s["bits"])
    view = fl.view_struct(synth.orbit_view(s["dims"], 0.7, 0.3, W, H, fovy_deg=4.0))
    opts = fl.render_opts()
    whole, rgba = (torch.full((H, W, 4), 7.0, device="cuda") for _ in range(2))
    stats, _ = fl.fhash_render(s["idx"], s["mlp"], s["tab_d"], s["prm_d"], bits, s["dims"], view,
                               2.5, s["tf_d"], W, H, opts, whole)
    ws = torch.empty(fl.fhash_render_state_bytes(W, H, s["dims"]), dtype=torch.uint8,
                     device="cuda")
    st = fl.fhash_render_begin(view, 2.5, W, H, bits, s["dims"], ws, rgba)
    assert st.n_alive == W * H
    pos, y = torch.empty(W * H, 4, device="cuda"), torch.empty(W * H, device="cuda")
    while st.n_alive > 0:
        pace = fl.fhash_render_pace(W * H, st.n_alive, opts.arm_max)
        ns = fl.fhash_render_march(st, opts, pace, pos, W * H)
        if ns:
            fl.fhash_fused_fwd(s["idx"], s["mlp"], pos[:ns], ns, s["tab_d"], s["prm_d"], y)
        fl.fhash_render_composite(st, y, s["tf_d"], opts, rgba)
    assert (stats.samples, stats.iterations) == (st.samples, st.iterations)
    np.testing.assert_array_equal(whole.cpu().numpy(), rgba.cpu().numpy())
