"""Levels of a few vertices, whose gradient every call sums in LDS before its
atomics: the separate adjoint and the fused backward against the FP64 oracle
(FP32 rule |gpu - oracle| <= 1e-5 mag + 1e-12), at batches around the chunk
sizes and around the rule's edge (a level joins at as many samples as vertices),
dense, active and hashed, with paired gradients and touched-segment flags."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2507_03836_amd import synth

pytestmark = pytest.mark.gpu

RES = [[2, 2, 2, 2], [5, 4, 3, 2], [9, 8, 6, 3]]  # 16, 120 and 1296 vertices
RTOL, ATOL = 1e-5, 1e-12


@pytest.fixture(scope="module")
def fl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    return fl


def _index(fl, kind, F):
    grid = fl.grid_desc(RES, F)
    if kind == "active":
        m = np.zeros((4, 7, 9, 11), np.uint8)
        m[1:3, 2:6, 1:7, 3:9] = 1
        bits = torch.from_numpy(synth.pack_mask_rows(m).view(np.int64)).cuda()
        idx, _, keep, _ = fl.fhash_build_index(grid, bits, list(m.shape[::-1]))
        return idx, O.Grid(np.array(RES), F, m), keep
    if kind == "hash":
        return fl.fhash_hash_index(grid, 6)[0], O.Grid(np.array(RES), F, hash_bits=6), None
    return fl.fhash_dense_index(grid)[0], O.Grid(np.array(RES), F), None


@pytest.mark.parametrize("n", [15, 16, 119, 257, 2049, 4096])
@pytest.mark.parametrize("kind", ["active", "dense", "hash"])
@pytest.mark.parametrize("F", [1, 2, 4, 8])
def test_encode_bwd_against_oracle(fl, F, kind, n):
    idx, g, _keep = _index(fl, kind, F)
    rng = np.random.default_rng(n + F)
    pos = rng.random((n, 4)).astype(np.float32)
    d = rng.uniform(-1, 1, (n, len(RES) * F)).astype(np.float32)
    ref, mag = O.encode_bwd(g, pos, d.astype(np.float64))
    dt = torch.zeros(g.total_slots * F, device="cuda")
    seg = (dt.numel() + 15) // 16
    flags = torch.zeros(seg, dtype=torch.uint8, device="cuda")
    fl.fhash_encode_bwd(idx, torch.from_numpy(pos).cuda(), n, torch.from_numpy(d).cuda(), dt,
                        touch=fl.touch_desc(flags, 0, dt.numel()))
    got = dt.cpu().numpy()
    err = np.abs(got.reshape(ref.shape).astype(np.float64) - ref)
    assert (err <= RTOL * mag + ATOL).all(), float((err - RTOL * mag).max())
    nz = np.pad(got, (0, seg * 16 - got.size)).reshape(seg, 16).any(1)
    assert not (nz & (flags.cpu().numpy() == 0)).any()  # every written segment is flagged


@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("kind", ["active", "dense"])
@pytest.mark.parametrize("F", [1, 2, 4])
def test_fused_bwd_against_oracle(fl, F, kind, paired):
    idx, g, _keep = _index(fl, kind, F)
    n, width = 1301, [len(RES) * F, 32, 32, 1]
    rng = np.random.default_rng(40 + F)
    pos = rng.random((n, 4)).astype(np.float32)
    dy = rng.uniform(-1, 1, n).astype(np.float32)
    table = rng.uniform(-1, 1, (g.total_slots, F)).astype(np.float32)
    params = synth.mlp_init(width, seed=9)
    enc, emag = O.encode_fwd(g, pos, table.astype(np.float64))
    _, acts, _ = O.mlp_fwd(width, params.astype(np.float64), enc, x_mag=emag)
    dp_ref, denc, dp_mag, denc_mag = O.mlp_bwd(width, params.astype(np.float64), acts,
                                               dy.reshape(-1, 1).astype(np.float64), n,
                                               dy_mag=np.abs(dy).reshape(-1, 1).astype(np.float64),
                                               x_mag=emag)
    dt_ref, _ = O.encode_bwd(g, pos, denc)
    _, dt_mag = O.encode_bwd(g, pos, denc_mag)
    runs = (g.total_slots * F + 15) // 16
    dt = torch.zeros(runs * 32 if paired else runs * 16, device="cuda")
    dp = torch.zeros(params.size, device="cuda")
    fl.fhash_fused_bwd(idx, fl.mlp_desc(width), torch.from_numpy(pos).cuda(), n,
                       torch.from_numpy(table.reshape(-1)).cuda(),
                       torch.from_numpy(params).cuda(), torch.from_numpy(dy).cuda(), dt, dp,
                       flags=fl.GRAD_PAIRED if paired else 0)
    got = dt.view(runs, -1)[:, :16].reshape(-1)[: g.total_slots * F].cpu().numpy()
    err = np.abs(got.reshape(dt_ref.shape).astype(np.float64) - dt_ref)
    assert (err <= RTOL * dt_mag + ATOL).all(), float((err - RTOL * dt_mag).max())
    err = np.abs(dp.cpu().numpy().astype(np.float64) - dp_ref)
    assert (err <= RTOL * dp_mag + ATOL).all()
    if paired:  # the gaps are not written
        assert not dt.view(runs, 32)[:, 16:].any()
