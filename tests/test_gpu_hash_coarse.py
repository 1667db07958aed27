"""The LDS scatter of a hashed index, which only FHASH_COARSE_LDS and
FHASH_SAMPLES_SORTED ask for: fused training and backward against the FP64 oracle on
sorted batches, whose vertex boxes fit the LDS image, and on batches in draw order,
where a chunk's box is the whole level and one level (39,546 floats at F = 2) is past
the image, so that its samples are added directly."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_hash import _close, _params, fl  # noqa: F401

pytestmark = pytest.mark.gpu

RES = [[4, 4, 4, 2], [8, 8, 8, 3], [13, 13, 13, 9]]  # 27, 686 and 13,824 cells
BITS = 9  # levels 1 and 2 hash into 512 rows


def _ws_bytes(fl, idx, mlp, n, flags):
    fake, nb = C.c_void_p(1 << 20), C.c_size_t(0)
    rc = fl.lib().fhash_fused_train(
        C.byref(idx), C.byref(mlp), fake, fake, C.c_int64(n), fake, fl.F32, fake, None,
        C.c_float(1.0), fake, fake, None, C.c_uint32(flags), None, None, C.byref(nb), None)
    assert rc == fl.OK, fl.lib().fhash_last_error()
    return nb.value


@pytest.mark.parametrize("flag,order", [("COARSE_LDS", "draw"), ("COARSE_LDS", "sorted"),
                                        ("SAMPLES_SORTED", "sorted")])
@pytest.mark.parametrize("F", [1, 2, 4])
def test_against_oracle(fl, F, flag, order):  # noqa: F811
    flags, n = getattr(fl, flag), 15007
    idx, _ = fl.fhash_hash_index(fl.grid_desc(RES, F), BITS)
    g = O.Grid(np.array(RES), F, hash_bits=BITS)
    rng = np.random.default_rng(50 + F)
    width = [len(RES) * F, 32, 32, 1]
    mlp = fl.mlp_desc(width)
    extra = _ws_bytes(fl, idx, mlp, n, flags) - (_ws_bytes(fl, idx, mlp, n, 0) + 255) // 256 * 256
    assert extra == len(RES) * n * F * 4  # every level takes the LDS scatter
    table = rng.uniform(-1, 1, (g.total_slots, F)).astype(np.float32)
    params = _params(width, 60 + F)
    pd = torch.from_numpy(rng.uniform(0, 1, (n, 4)).astype(np.float32)).cuda()
    td = torch.from_numpy(rng.uniform(0, 1, n).astype(np.float32)).cuda()
    if order == "sorted":
        fl.fhash_sort_samples(pd, td, n)
    pos, tgt = pd.cpu().numpy(), td.cpu().numpy()
    tab, prm = torch.from_numpy(table).cuda(), torch.from_numpy(params).cuda()
    e_ref, e_mag = O.encode_fwd(g, pos, table.astype(np.float64))
    y, acts, ymag = O.mlp_fwd(width, params.astype(np.float64), e_ref, x_mag=e_mag)
    _, dy = O.mse(y[:, 0], tgt.astype(np.float64))
    for call in ("train", "bwd"):
        if call == "train":
            d, dm = dy.reshape(-1, 1), 2.0 * (ymag + np.abs(tgt)[:, None]) / n
        else:
            dyd = torch.from_numpy(rng.uniform(-1, 1, n).astype(np.float32)).cuda()
            d = dyd.cpu().numpy().astype(np.float64).reshape(-1, 1)
            dm = np.abs(d)
        dp_ref, denc, dpm, dencm = O.mlp_bwd(width, params.astype(np.float64), acts, d, n,
                                             dy_mag=dm, x_mag=e_mag)
        dt_ref, _ = O.encode_bwd(g, pos, denc)
        _, dtm = O.encode_bwd(g, pos, dencm)
        dt = torch.zeros(g.total_slots, F, device="cuda")
        dp = torch.zeros(len(params), device="cuda")
        if call == "train":
            fl.fhash_fused_train(idx, mlp, pd, td, n, tab, prm, dt, dp, flags=flags)
        else:
            fl.fhash_fused_bwd(idx, mlp, pd, n, tab, prm, dyd, dt, dp, flags=flags)
        _close(dt.cpu().numpy(), dt_ref, dtm, f"{call} d_table")
        _close(dp.cpu().numpy(), dp_ref, dpm, f"{call} d_params")
