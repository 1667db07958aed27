"""The decoder gradient of the fused backward under contention: integer weights,
inputs and output gradients, so that every sum is exact in FP32 in any order and
an add that the waves of a workgroup lose between them shows.  The reference is
the same network on whole numbers in FP64; the sums' magnitudes are held below 2^24."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

L, F = 16, 2
RES = [[3, 3, 3, 3]] * L  # cells of 0.5; positions 0.25 and 0.75 are cell centres


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


def _sparse(rng, shape):
    return rng.integers(-1, 2, shape) * (rng.random(shape) < 0.2)


def _reference(cell, table, layers, dy):
    """(y, parameter gradient, its term magnitudes) in integers; layers: (W, b)."""
    corner = np.stack(np.meshgrid(*[[0, 1]] * 4, indexing="ij"), -1).reshape(-1, 4)
    v = cell[:, None, :] + corner[None]                       # x, y, z, t
    row = ((v[..., 3] * 3 + v[..., 2]) * 3 + v[..., 1]) * 3 + v[..., 0]
    x = np.concatenate([table[l][row].sum(1) for l in range(L)], 1)  # 16 x / 16
    acts = [x]
    for W, b in layers[:-1]:
        acts.append(np.maximum(acts[-1] @ W.T + b, 0))
    W, b = layers[-1]
    y = (acts[-1] @ W.T + b)[:, 0]
    out, mag, d = [], [], dy[:, None]
    for k in range(len(layers) - 1, -1, -1):
        out = [(d.T @ acts[k]).ravel(), d.sum(0)] + out
        mag = [(np.abs(d).T @ np.abs(acts[k])).ravel(), np.abs(d).sum(0)] + mag
        if k:
            d = (d @ layers[k][0]) * (acts[k] > 0)
    return y, np.concatenate(out), np.concatenate(mag)


@pytest.mark.parametrize("dt", ["f32", "f16"])
@pytest.mark.parametrize("hidden,nh", [(32, 2), (64, 3)])
@pytest.mark.parametrize("n", [4096 + 7, 70001])
def test_no_add_is_lost(fl, n, hidden, nh, dt):
    rng = np.random.default_rng(n + hidden + nh)
    cell = rng.integers(0, 2, (n, 4))
    table = [_sparse(rng, (81, F)).astype(np.float64) for _ in range(L)]
    width = [L * F] + [hidden] * nh + [1]
    layers = [(_sparse(rng, (o, i)).astype(np.float64), _sparse(rng, (o,)).astype(np.float64))
              for i, o in zip(width, width[1:])]
    layers[-1][0][:, ::2] = 1
    dy = rng.integers(-1, 2, n).astype(np.float64)
    y, ref, mag = _reference(cell, table, layers, dy)
    assert mag.max() < 2 ** 24 and np.abs(y).max() < 2 ** 24 and (ref != 0).sum() > ref.size // 8
    idx = fl.fhash_dense_index(fl.grid_desc(RES, F))[0]
    mlp = fl.mlp_desc(width, {"f32": fl.F32, "f16": fl.F16}[dt])
    params = np.concatenate([p.ravel() for layer in layers for p in layer]).astype(np.float32)
    pos = torch.from_numpy((0.25 + 0.5 * cell).astype(np.float32)).cuda()
    tab = torch.from_numpy(16.0 * np.concatenate(table).astype(np.float32)).cuda()
    prm = torch.from_numpy(params).cuda()
    dyd = torch.from_numpy(dy.astype(np.float32)).cuda()
    dtab, dprm = torch.zeros_like(tab), torch.zeros_like(prm)
    out = torch.empty(n, device="cuda")
    fl.fhash_fused_fwd(idx, mlp, pos, n, tab, prm, out)
    assert np.array_equal(out.cpu().numpy(), y)
    fl.fhash_fused_bwd(idx, mlp, pos, n, tab, prm, dyd, dtab, dprm)
    assert np.array_equal(dprm.cpu().numpy(), ref)
