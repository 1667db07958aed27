"""The fused calls at the sizes where their launch changes shape: waves per
workgroup go from 1 to 8 as a batch grows to 2048 blocks of 16 samples.  A
sample's output does not depend on the batch it came in, bit for bit; gradients
against the FP64 oracle (|gpu - oracle| <= 1e-5 mag + 1e-12) either side of the
first change."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu

RES = [[6, 5, 4, 3], [12, 10, 9, 4], [25, 21, 18, 7]]
RTOL, ATOL = 1e-5, 1e-12


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


@pytest.mark.parametrize("dtype,hidden,layers", [("f32", 32, 1), ("f32", 64, 3), ("f16", 64, 2),
                                                 ("bf16", 32, 3)])
def test_outputs_do_not_depend_on_the_batch(fl, dtype, hidden, layers):
    F, width = 2, [len(RES) * 2] + [hidden] * layers + [1]
    idx, _ = fl.fhash_dense_index(fl.grid_desc(RES, F))
    rows = int(idx.slot_offset[len(RES)])
    rng = np.random.default_rng(11)
    table = torch.from_numpy(rng.uniform(-1, 1, rows * F).astype(np.float32)).cuda()
    params = torch.from_numpy(synth.mlp_init(width, seed=4)).cuda()
    mlp = fl.mlp_desc(width, {"f32": fl.F32, "f16": fl.F16, "bf16": fl.BF16}[dtype])
    pos = torch.from_numpy(rng.random((32785, 4)).astype(np.float32)).cuda()

    def out(p):
        y = torch.full((p.shape[0],), float("nan"), device="cuda")
        fl.fhash_fused_fwd(idx, mlp, p, p.shape[0], table, params, y)
        return y

    whole = out(pos)
    assert torch.isfinite(whole).all()
    for n in (1, 15, 16, 17, 4095, 4096, 4097, 8193, 12289, 28672, 28673, 32768, 32769):
        torch.testing.assert_close(out(pos[:n]), whole[:n], rtol=0, atol=0)


@pytest.mark.parametrize("n", [1, 16, 17, 4096, 4097])
@pytest.mark.parametrize("F,hidden,layers", [(1, 32, 2), (2, 64, 3), (4, 64, 1)])
def test_fused_bwd_against_oracle(fl, F, hidden, layers, n):
    width = [len(RES) * F] + [hidden] * layers + [1]
    idx, _ = fl.fhash_dense_index(fl.grid_desc(RES, F))
    g = O.Grid(np.array(RES), F)
    rng = np.random.default_rng(20 + n)
    pos = rng.random((n, 4)).astype(np.float32)
    dy = rng.uniform(-1, 1, n).astype(np.float32)
    table = rng.uniform(-1, 1, (g.total_slots, F)).astype(np.float32)
    params = synth.mlp_init(width, seed=5)
    p64, dy64 = params.astype(np.float64), dy.reshape(-1, 1).astype(np.float64)
    enc, emag = O.encode_fwd(g, pos, table.astype(np.float64))
    _, acts, _ = O.mlp_fwd(width, p64, enc, x_mag=emag)
    dp_ref, denc, dp_mag, denc_mag = O.mlp_bwd(width, p64, acts, dy64, n, dy_mag=np.abs(dy64),
                                               x_mag=emag)
    dt_ref, _ = O.encode_bwd(g, pos, denc)
    _, dt_mag = O.encode_bwd(g, pos, denc_mag)
    dt = torch.zeros(g.total_slots * F, device="cuda")
    dp = torch.zeros(params.size, device="cuda")
    fl.fhash_fused_bwd(idx, fl.mlp_desc(width), torch.from_numpy(pos).cuda(), n,
                       torch.from_numpy(table.reshape(-1)).cuda(),
                       torch.from_numpy(params).cuda(), torch.from_numpy(dy).cuda(), dt, dp)
    err = np.abs(dt.cpu().numpy().reshape(dt_ref.shape).astype(np.float64) - dt_ref)
    assert (err <= RTOL * dt_mag + ATOL).all(), float((err - RTOL * dt_mag).max())
    err = np.abs(dp.cpu().numpy().astype(np.float64) - dp_ref)
    assert (err <= RTOL * dp_mag + ATOL).all(), float((err - RTOL * dp_mag).max())
