"""The dense Adam sweep over the layout with the moments beside the parameters
against separate arrays, bit for bit: counts either side of whole blocks of 16
and of the 32 blocks a wave takes together, FP16 and BF16 shadows, a skipped
step, touched-segment flags (the gradient is zero wherever unflagged)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


@pytest.mark.parametrize("n", [3, 16, 17, 100, 511, 512, 513, 16 * 129 + 4, 70001])
@pytest.mark.parametrize("mode", ["plain", "f16", "bf16", "skip", "touch"])
def test_equal_to_separate_arrays(fl, n, mode):
    rng = np.random.default_rng(n)
    nb = (n + 15) // 16
    g = rng.normal(size=nb * 16).astype(np.float32) * 1e-3
    g[n:] = 0
    seg = rng.random(nb) < 0.4
    if mode == "touch":
        g = np.where(np.repeat(seg, 16), g, 0).astype(np.float32)
    g[::7] = 0
    arrays = {"p": rng.normal(size=nb * 16), "m": rng.normal(size=nb * 16) * 1e-3,
              "v": rng.random(nb * 16) * 1e-6, "g": g}
    dev = {k: torch.from_numpy(np.asarray(a, np.float32)).cuda() for k, a in arrays.items()}
    pm = torch.stack([dev["p"].view(-1, 16), dev["m"].view(-1, 16)], 1).reshape(-1).contiguous()
    gv = torch.stack([dev["g"].view(-1, 16), dev["v"].view(-1, 16)], 1).reshape(-1).contiguous()
    opt = fl.AdamDesc()
    opt.lr, opt.beta1, opt.beta2, opt.eps, opt.step, opt.grad_scale = 0.01, 0.9, 0.999, 1e-8, 7, 0.5
    dt = {"f16": torch.float16, "bf16": torch.bfloat16}.get(mode)
    sh = [torch.zeros(n + 8, dtype=dt, device="cuda") for _ in range(2)] if dt else [None, None]
    inf = torch.ones(1, dtype=torch.int32, device="cuda") if mode == "skip" else None
    flags = [torch.from_numpy(seg.astype(np.uint8)).cuda() for _ in range(2)]
    begin = 16 if n >= 32 else 0
    touch = [fl.touch_desc(f, begin, n) if mode == "touch" else None for f in flags]
    if mode == "touch" and begin:
        flags[0][0] = flags[1][0] = 1  # before `begin`: not looked at, not cleared
    opt.moments = fl.MOMENTS_SEPARATE
    fl.fhash_step(opt, dev["p"], dev["g"], dev["m"], dev["v"], shadow=sh[0], found_inf=inf,
                  touch=touch[0], n=n)
    opt.moments = fl.MOMENTS_WITH_PARAMS
    fl.fhash_step(opt, pm, gv, pm[16:], gv[16:], shadow=sh[1], found_inf=inf, touch=touch[1], n=n)
    got = {"p": pm.view(-1, 2, 16)[:, 0], "m": pm.view(-1, 2, 16)[:, 1],
           "g": gv.view(-1, 2, 16)[:, 0], "v": gv.view(-1, 2, 16)[:, 1]}
    for k, x in got.items():
        torch.testing.assert_close(x.reshape(-1), dev[k], rtol=0, atol=0, msg=k)
    assert not dev["g"][:n].any()
    if dt:
        torch.testing.assert_close(sh[1], sh[0], rtol=0, atol=0)
    if mode == "touch":
        torch.testing.assert_close(flags[1], flags[0], rtol=0, atol=0)
