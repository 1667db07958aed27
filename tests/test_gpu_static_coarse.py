"""fhash_fused_train_static with levels of a few vertices, which go through the LDS
scatter in pieces of the batch: around the size of a piece (131,072 samples for 32
decoder inputs), with and without FHASH_SAMPLES_SORTED, on integer networks whose
sums are exact in FP32, so that gradients and loss equal the reference and those of
the call with a workspace bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

from test_gpu_decoder_grad_exact import F, L, RES, _reference, _sparse, fl  # noqa: F401

pytestmark = pytest.mark.gpu

PIECE = (1 << 22) // (L * F)


def _static(fl, idx, mlp, pos, tgt, n, tab, prm, scale, dt, dp, loss, flags):
    P = C.c_void_p
    rc = fl.lib().fhash_fused_train_static(
        C.byref(idx), C.byref(mlp), P(pos.data_ptr()), P(tgt.data_ptr()), C.c_int64(n),
        P(tab.data_ptr()), fl.F32, P(prm.data_ptr()), None, C.c_float(scale), P(dt.data_ptr()),
        P(dp.data_ptr()), P(loss.data_ptr()), C.c_uint32(flags), None,
        P(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, fl.lib().fhash_last_error()


@pytest.mark.parametrize("sorted_", [False, True])
@pytest.mark.parametrize("dt", ["f32", "f16"])
@pytest.mark.parametrize("n", [80, 81, 5003, PIECE, PIECE + 1, 2 * PIECE + 1234])
def test_static_call_in_pieces(fl, n, dt, sorted_):
    rng = np.random.default_rng(n)
    width = [L * F, 32, 32, 1]
    table = [_sparse(rng, (81, F)).astype(np.float64) for _ in range(L)]
    layers = [(_sparse(rng, (o, i)).astype(np.float64), _sparse(rng, (o,)).astype(np.float64))
              for i, o in zip(width, width[1:])]
    layers[-1][0][:, ::2] = 1
    cell = rng.integers(0, 2, (n, 4))
    if sorted_:
        cell = cell[np.lexsort(cell.T)]
    y = _reference(cell, table, layers, np.zeros(n))[0]
    dy = rng.integers(-1, 2, n).astype(np.float64)
    _, ref, mag = _reference(cell, table, layers, dy)
    assert mag.max() < 2 ** 24
    idx = fl.fhash_dense_index(fl.grid_desc(RES, F))[0]
    mlp = fl.mlp_desc(width, {"f32": fl.F32, "f16": fl.F16}[dt])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    pos, tgt = dev(0.25 + 0.5 * cell), dev(y - dy)
    tab = dev(16.0 * np.concatenate(table))
    prm = dev(np.concatenate([p.ravel() for layer in layers for p in layer]))
    flags = fl.SAMPLES_SORTED if sorted_ else 0
    out = []
    for static in (True, False):
        dtab, dprm = torch.zeros_like(tab), torch.zeros_like(prm)
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        if static:
            _static(fl, idx, mlp, pos, tgt, n, tab, prm, n / 2, dtab, dprm, loss, flags)
        else:
            fl.fhash_fused_train(idx, mlp, pos, tgt, n, tab, prm, dtab, dprm, loss, n / 2,
                                 flags=flags)
        assert np.array_equal(dprm.cpu().numpy(), ref)
        assert loss.item() == (dy ** 2).sum()
        out.append(dtab.cpu().numpy())
    assert np.array_equal(out[0], out[1]) and np.abs(out[0]).sum() > 0
